// Householder tridiagonalisation of a symmetric matrix (first step of the
// spectral decomposition used by Alg. 3).
//
// The trailing matrix lives in registers, one lower-triangular tile per
// workgroup of a cooperative launch, and is updated there (A -= v w^T + w v^T,
// summed apart and rounded into the tile once per kFlush or kLazy columns, see
// Tile), with ONE exchange per column.  For column j with
// sub-column u (rows j+1..n-1) the reflector is v = (u - beta e1) c, c =
// 1/(alpha - beta).  Everything the column needs from v is linear in v, so
// before the exchange each workgroup forms its tile's share of the product
// with the *unnormalised* u (A u and, off the diagonal, A^T u), its share of
// u^T A u and ||u||^2, and publishes column j+1 of its tile.  After the
// exchange every workgroup finishes the scalars, y = A v, w = tau y -
// (tau/2)(tau y^T v) v and the next column u' = A(:, j+1) - v w_{j+1} - w for
// the rows of its tile, and updates the tile.  A launch reduces kLaunchCols
// columns, then writes its tiles back; the next one cuts the smaller trailing
// matrix anew.  The last kTailRows rows take one workgroup (sytrd_tail_kernel).
//
// The exchange.  Small tiles (kTag): every word carries its column's tag, so
// the reads that gather it are the wait; the scalars from every workgroup
// also say that all have read the words of the column before, whose buffer
// the next column takes.  Words go out twice as wide and are read again until
// they are there, so larger tiles, which read more, exchange plain values
// around a grid barrier.  Measured with tags and with the barrier: n = 1000
// 3.4 and 4.2 ms, n = 1531 6.3 and 7.2 (64-row tiles); n = 4096, whose first
// launches have 192- and 128-row tiles, 26.3 and 23.7 (24.5 with kLazy in the
// kernel, which changed the order of its instructions).  Each workgroup's
// scalars have a 64-byte line of their own: packed together they took 0.4 ms
// longer at n = 1000.
//
// What bounds it: the latency of a column, 4.1 us at n = 1531, of which the
// exchange is about half and the instructions of product, row work and update
// the rest.  (A blocked panel that left the matrix alone for 32 columns and
// corrected every column with V and W spent 9.3 us per column at n = 1531 and
// 9.8 at n = 4096: its row corrections, V^T u, W^T u and their exchange cost
// more than the update of the register tile.  Now 4.1 and 6.0 us, 14.3 -> 6.3
// ms and 40.2 -> 24.5 ms, with an X_0 that is 5 % closer to the root.)
#include <algorithm>
#include <vector>

#include "gridsync.hpp"
#include "kernels.hpp"
#include "profile.hpp"
#include "tridiag.hpp"

namespace msqrt {

namespace {

constexpr int kTRMax = 22;    // max tiles per dimension: 253 workgroups, one per CU
constexpr int kGMax = kTRMax * (kTRMax + 1) / 2;
constexpr int kMaxN = kTRMax * 192 + 1;  // largest order
constexpr int kLaunchCols = 128;  // n = 4096: 27.6, 26.0, 25.3, 25.0 ms for 32, 64, 128, 256 (without kDelta and tags)
constexpr int kFlush = 32;    // columns between flushes of the accumulated updates

// How the panel kernel is built for tiles of 64 RPL rows: threads, and how a
// tile's updates are kept from rounding it at every column (which doubled the
// error of X_0 at n = 4096, kappa = 1e4: 1.9e-6 to 4.0e-6).  kDelta: they are
// summed in registers beside the tile, where those hold both: 1024 threads have
// 128 registers each, 512 have 256.  Otherwise the last up to kLazy columns'
// v and w wait in LDS, the product and the published column are corrected by
// them, and the tile is updated once for all of them.  (With one rounding per
// column in these tiles X_0 was 16 % worse for 64 x 512 and, in double, 9 % at
// n = 4096 than with panels of 32 columns, and the gradient of 64 x 512 1.7
// times; now they are 0.90, 1.00 and 0.78 of it.  It costs 0.25 ms of the 64 x
// 512 reduction, 2.04 -> 2.29, and 1.6 of 28.5 ms at n = 4096 in double.)
// kTag: the exchange is by tagged words.
constexpr int kLazy = 8;
template <typename T, int RPL>
struct Tile;
template <> struct Tile<float, 1> { static constexpr int NT = 1024; static constexpr bool kDelta = true; static constexpr bool kTag = true; };
template <> struct Tile<float, 2> { static constexpr int NT = 1024; static constexpr bool kDelta = true; static constexpr bool kTag = false; };
template <> struct Tile<float, 3> { static constexpr int NT = 512; static constexpr bool kDelta = true; static constexpr bool kTag = false; };
template <> struct Tile<float, 4> { static constexpr int NT = 1024; static constexpr bool kDelta = false; static constexpr bool kTag = false; };
template <> struct Tile<double, 1> { static constexpr int NT = 1024; static constexpr bool kDelta = true; static constexpr bool kTag = true; };
template <> struct Tile<double, 2> { static constexpr int NT = 512; static constexpr bool kDelta = true; static constexpr bool kTag = false; };
template <> struct Tile<double, 3> { static constexpr int NT = 512; static constexpr bool kDelta = false; static constexpr bool kTag = false; };
template <> struct Tile<double, 4> { static constexpr int NT = 1024; static constexpr bool kDelta = false; static constexpr bool kTag = false; };

template <typename T>
struct PanelArgs {
  int n, p, nc;  // matrix size, first column, columns of this launch
  int TR, ts;    // tiles per dimension over the rows p .. n - 1, tile size
  T* A;          // n x n, ld n (lower triangle read and kept)
  T* d;
  T* e;
  T* tau;
  // the exchanged words (tag: the column's) of batch entry 0; sX per entry
  tword* x;
  unsigned* bar;  // barrier words of batch entry 0; the failure flag is among them
  BarrierBase bar_base;
  // batch entry b = blockIdx.y: every pointer above advances by b strides
  int64_t sA, sD, sX;
};

// The exchanged words of one entry, two buffers (column parity): partial
// products [TR][n], column j + 1 [n], alpha; u^T A u per workgroup and wave of
// the rows of I, ||u||^2 per diagonal workgroup and wave.
template <typename T>
struct Exchange {
  static constexpr int W = kTagW<T>;
  int64_t yp, cl, al, s0, s1, size;  // offsets in a buffer
  __host__ __device__ Exchange(int n, int TR) {
    yp = 0;
    cl = (int64_t)TR * n * W;
    al = cl + (int64_t)n * W;
    s0 = al + W;
    s1 = s0 + (int64_t)TR * (TR + 1) / 2 * 8;  // up to 4 doubles of 2 words
    size = s1 + (int64_t)TR * 8;
  }
};

// a + b after the halves (the rows of 16 lanes) of the wave have been exchanged:
// lanes of the first half (even rows) get a summed over both, the others b.
__device__ inline float swap_add32(float a, float b) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ inline float swap_add16(float a, float b) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ inline double join(unsigned lo, unsigned hi) {
  return __longlong_as_double(((long long)hi << 32) | lo);
}
__device__ inline double swap_add32(double a, double b) {
  const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto l = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return join(l[0], h[0]) + join(l[1], h[1]);
}
__device__ inline double swap_add16(double a, double b) {
  const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto l = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return join(l[0], h[0]) + join(l[1], h[1]);
}

// The reflector and the product w of one column from its sums: alpha =
// u_{j+1}, sig = ||u_{j+2..}||^2, uAu = u^T A u, y1 and a11 = entries j+1 of
// A u and of column j+1.  A column of norm below 1e-140 (the matrix is scaled to
// about 1) counts as reduced: its squares underflow and 1 / |u|^2 overflows.
struct Reflector {
  double beta, tau, c, wv;  // wv = tau v^T A v
  __device__ Reflector(double alpha, double sig, double uAu, double y1, double a11) {
    beta = alpha;
    tau = c = 0.0;
    if (sig != 0.0 && alpha * alpha + sig > 1e-280) {
      beta = -copysign(sqrt(alpha * alpha + sig), alpha);
      tau = (beta - alpha) / beta;
      c = 1.0 / (alpha - beta);
    }
    wv = tau * c * c * (uAu - 2.0 * beta * y1 + beta * beta * a11);
  }
  // w_i from (A u)_i, column entry a_i and v_i
  __device__ double w(double y, double a, double v) const { return tau * (c * (y - beta * a)) - 0.5 * tau * wv * v; }
};

template <typename T, int RPL>
__global__ __launch_bounds__((Tile<T, RPL>::NT)) void sytrd_panel_kernel(PanelArgs<T> a) {
  constexpr int NT = Tile<T, RPL>::NT, NW = NT / kWave;
  constexpr bool kDelta = Tile<T, RPL>::kDelta;
  constexpr int PB = kDelta ? 1 : kLazy;  // columns of v and w in LDS
  constexpr int TS = kWave * RPL, CW = TS / NW, CQ = CW / 4;  // tile size, columns per wave and lane row
  // Row work of a column: rows of I on threads [0, TS), rows of K on
  // [NT / 2, NT / 2 + TS); the partial sums of the scalars of kScN workgroups
  // per thread on the waves between them; the pivot row on kPivT.
  constexpr int kKT = NT / 2, kScN = NT == 1024 ? 1 : 2, kPivT = NT == 1024 ? 768 : NT - 1;
  static_assert(NT == 1024 ? TS <= 256 : NT == 512 && TS <= 192, "thread ranges");
  const int n = a.n, TR = a.TR, G = TR * (TR + 1) / 2;
  // workgroup (x, y) = (tile, batch entry); both ids and all that is derived
  // from them are scalar
  {
    const int64_t bz = blockIdx.y;
    a.A += bz * a.sA;
    a.d += bz * a.sD;
    a.e += bz * a.sD;
    a.tau += bz * a.sD;
    a.x += bz * a.sX;
    a.bar += bz * kBarWords;
  }
  const int blk = blockIdx.x;
  // tile (bi, bj) of the lower triangle, row-major: bi (bi + 1) / 2 <= blk
  int bi = 0;
  while ((bi + 1) * (bi + 2) / 2 <= blk) ++bi;
  const int bj = blk - bi * (bi + 1) / 2;
  const bool diag = bi == bj, offdiag = !diag;
  unsigned sub_base = 0;
#pragma unroll
  for (int g = 0; g < 8; ++g)
    if (g == (blk & 7)) sub_base = a.bar_base.sub[g];
  unsigned* const fail = a.bar + kBarFail;
  const Exchange<T> ex(n, TR);
  constexpr int W = Exchange<T>::W;
  constexpr bool kTag = Tile<T, RPL>::kTag;
  constexpr int kCh = sizeof(T) == 8 ? 6 : 8;  // partial products read at a time
  const int p = a.p;
  const int I0 = p + bi * a.ts, nI = max(0, min(n - I0, a.ts));
  const int K0 = p + bj * a.ts, nK = max(0, min(n - K0, a.ts));
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), cb = wave * CW;
  const unsigned ld = (unsigned)n;  // n^2 < 2^31: 32-bit offsets
  T* A = a.A;
  __shared__ __attribute__((aligned(16))) T uI[TS], uK[TS], vw[PB][4][TS];  // vw: v and w of the rows of I, of K
  __shared__ T zred[NW][TS], zK[TS], dots[4][PB];
  __shared__ double red[2][4];
  __shared__ T piv[3];  // alpha, y_{j+1}, A(j+1, j+1)
  const bool rowI = tid < nI, rowK = offdiag && tid >= kKT && tid - kKT < nK;

  T v[CW][RPL], dl[kDelta ? CW : 1][kDelta ? RPL : 1];  // the tile is v - dl
  auto entry = [&](int c, int q) -> T {
    if constexpr (kDelta) return v[c][q] - dl[c][q];
    else return v[c][q];
  };
#pragma unroll
  for (int c = 0; c < CW; ++c)
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
      const int r = lane + q * kWave, k = cb + c;
      const int row = I0 + r, col = K0 + k;
      if constexpr (kDelta) dl[c][q] = T(0);
      v[c][q] = (r < nI && k < nK) ? A[max(row, col) + (unsigned)min(row, col) * ld] : T(0);
    }
  if (tid < TS) uI[tid] = (rowI && I0 + tid > p) ? A[I0 + tid + (unsigned)p * ld] : T(0);
  if (tid >= kKT && tid - kKT < TS) uK[tid - kKT] = (tid - kKT < nK && K0 + tid - kKT > p) ? A[K0 + tid - kKT + (unsigned)p * ld] : T(0);
  if (p == 0 && blk == 0 && tid == 0) a.d[0] = A[0];
  if (tid < 8) red[tid / 4][tid % 4] = 0.0;
  __syncthreads();

  // kGroup columns, then the update of the tile that they left
  constexpr int kGroup = kDelta ? kFlush : kLazy;
#pragma clang loop unroll(disable)
  for (int g0 = 0; g0 < a.nc; g0 += kGroup) {
    const int g1 = min(g0 + kGroup, a.nc);
#pragma clang loop unroll(disable)
    for (int jj = g0; jj < g1; ++jj) {
      const int j = p + jj, buf = jj & 1;
      const unsigned tag = step_tag((unsigned)j);
      tword* const xb = a.x + buf * ex.size;
      tword* const yp = xb + ex.yp;
      tword* const cl = xb + ex.cl;
      T* const yv = reinterpret_cast<T*>(yp);  // the same without tags
      T* const cv = reinterpret_cast<T*>(cl);
      const int sl = kDelta ? 0 : jj - g0;  // slot of this column; the slots before it wait
      // column j + 1 as it is before this column's update
      const int kc = j + 1 - K0 - cb;
      if (kc >= 0 && kc < CW && j + 1 - K0 < nK) {
        T wait[RPL] = {};
        if constexpr (!kDelta) {
#pragma clang loop unroll(disable)
          for (int t = 0; t < sl; ++t) {
            const T vc = vw[t][2][cb + kc], wc = vw[t][3][cb + kc];
#pragma unroll
            for (int q = 0; q < RPL; ++q) wait[q] += vw[t][0][lane + q * kWave] * wc + vw[t][1][lane + q * kWave] * vc;
          }
        }
#pragma unroll
        for (int c = 0; c < CW; ++c)
          if (c == kc) {
#pragma unroll
            for (int q = 0; q < RPL; ++q) {
              const int r = lane + q * kWave;
              if (r < nI && I0 + r >= j + 1) {
                if constexpr (kTag) tag_store(cl + (unsigned)(I0 + r) * W, entry(c, q), tag);
                else cstore(cv + I0 + r, kDelta ? entry(c, q) : v[c][q] - wait[q]);
              }
            }
          }
      }
      // sums by which the waiting columns correct the products below: w_K^T u_K,
      // v_K^T u_K, w_I^T u_I, v_I^T u_I
      if constexpr (!kDelta) {
        for (int x = wave; x < (offdiag ? 4 : 2) * sl; x += NW) {
          const int kind = x / sl, t = x % sl;
          const T* a1 = vw[t][3 - kind];
          const T* a2 = kind < 2 ? uK : uI;
          T d = T(0);
#pragma unroll
          for (int q = 0; q < RPL; ++q) d += a1[lane + q * kWave] * a2[lane + q * kWave];
          d = wsum(d);
          if (lane == 0) dots[kind][t] = d;
        }
      }
      // partial products: rows (one sum per wave), columns off the diagonal
      {
        T zi[RPL], ui[RPL], zk[CW];
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
          zi[q] = T(0);
          ui[q] = uI[lane + q * kWave];
        }
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          const T uk = uK[cb + c];
          zk[c] = T(0);
#pragma unroll
          for (int q = 0; q < RPL; ++q) {
            const T x = entry(c, q);
            zi[q] += x * uk;
            zk[c] += x * ui[q];
          }
        }
#pragma unroll
        for (int q = 0; q < RPL; ++q) zred[wave][lane + q * kWave] = zi[q];
        if (offdiag) {
          // column sums over the 64 lanes by halving exchanges: lane row R ends
          // with columns CQ R .. CQ R + CQ - 1
          T z2[CW / 2], z4[CQ];
#pragma unroll
          for (int c = 0; c < CW / 2; ++c) z2[c] = swap_add32(zk[c], zk[c + CW / 2]);
#pragma unroll
          for (int c = 0; c < CQ; ++c) z4[c] = rsum16(swap_add16(z2[c], z2[c + CQ]));
          const int l16 = lane & 15;
          T z = z4[0];
#pragma unroll
          for (int c = 1; c < CQ; ++c) z = l16 == c ? z4[c] : z;
          if (l16 < CQ) zK[cb + CQ * (lane >> 4) + l16] = z;
        }
      }
      __syncthreads();
      double s0 = 0.0, s1 = 0.0;
      if (tid < TS) {
        T z = T(0);
#pragma unroll
        for (int w = 0; w < NW; ++w) z += zred[w][tid];
        if constexpr (!kDelta) {
          T wait = T(0);
#pragma clang loop unroll(disable)
          for (int t = 0; t < sl; ++t) wait += vw[t][0][tid] * dots[0][t] + vw[t][1][tid] * dots[1][t];
          z -= wait;
        }
        const double u = (double)uI[tid];
        if (rowI) {
          if constexpr (kTag) tag_store(yp + ((unsigned)bj * n + I0 + tid) * W, z, tag);
          else cstore(yv + (unsigned)bj * n + I0 + tid, z);
        }
        s0 = wsum(u * (double)z);
        s1 = diag ? wsum(I0 + tid >= j + 2 ? u * u : 0.0) : 0.0;
        if (offdiag) s0 *= 2.0;
        if (diag && rowI && I0 + tid == j + 1) tag_store(xb + ex.al, uI[tid], tag);
        if (lane == 0) {
          tword* const p0 = xb + ex.s0 + 8 * blk + 2 * wave;
          tword* const p1 = xb + ex.s1 + 8 * bi + 2 * wave;
          if constexpr (kTag) {
            tag_store(p0, s0, tag);
            if (diag) tag_store(p1, s1, tag);
          } else {
            cstore(reinterpret_cast<double*>(p0), s0);
            if (diag) cstore(reinterpret_cast<double*>(p1), s1);
          }
        }
      } else if (rowK) {
        const int r = tid - kKT;
        T z = zK[r];
        if constexpr (!kDelta) {
          T wait = T(0);
#pragma clang loop unroll(disable)
          for (int t = 0; t < sl; ++t) wait += vw[t][2][r] * dots[2][t] + vw[t][3][r] * dots[3][t];
          z -= wait;
        }
        if constexpr (kTag) tag_store(yp + ((unsigned)bi * n + K0 + r) * W, z, tag);
        else cstore(yv + (unsigned)bi * n + K0 + r, z);
      }
      if constexpr (!kTag) grid_barrier<NT>(a.bar, a.bar_base, sub_base, blk, G, jj + 1);
      // gather: all words of a thread are in flight together
      const bool pivot = tid == kPivT;
      const bool sums = NT == 1024 ? tid >= 256 && tid < 512 : (tid & 255) >= 192;
      const int swave = NT == 1024 ? wave - 4 : wave / 4, sidx = swave * kWave + lane;
      const int row = pivot ? j + 1 : rowI ? I0 + tid : (rowK ? K0 + tid - kKT : 0);
      const bool live = (rowI || rowK) && row >= j + 1;
      T y = T(0), a1 = T(0);
      if (kTag && (live || pivot)) {
        const unsigned stride = 8u * W * (unsigned)n;
        unsigned ro = 8u * W * (unsigned)row;
        asm volatile("" : "+v"(ro));  // the words' offsets are not kept over the columns
        {
          tword w[kCh * W + W];
          auto load = [&](int k) {
            if (k >= kCh * W) return tag_word(cl, ro + 8u * (k - kCh * W));
            return k / W < TR ? tag_word(yp, ro + (unsigned)(k / W) * stride + 8u * (k % W)) : (tword)tag << 32;
          };
          tag_load(w, load, tag, fail);
#pragma unroll
          for (int b = 0; b < kCh; ++b) y += tag_value<T>(w + b * W);
          a1 = tag_value<T>(w + kCh * W);
        }
        for (int b0 = kCh; b0 < TR; b0 += kCh) {
          tword w[kCh * W];
          auto load = [&](int k) {
            return b0 + k / W < TR ? tag_word(yp, ro + (unsigned)(b0 + k / W) * stride + 8u * (k % W)) : (tword)tag << 32;
          };
          tag_load(w, load, tag, fail);
#pragma unroll
          for (int b = 0; b < kCh; ++b) y += tag_value<T>(w + b * W);
        }
      }
      if constexpr (!kTag) {
        if (live || pivot) {
          T t[kTRMax];
#pragma unroll
          for (int b = 0; b < kTRMax; ++b) t[b] = b < TR ? cload(yv + (unsigned)b * n + row) : T(0);
          a1 = cload(cv + row);
#pragma unroll
          for (int b = 0; b < kTRMax; ++b) y += t[b];
        }
      }
      if (sums) {
        // the waves' sums of workgroup b (s0) and of diagonal workgroup b (s1)
        auto gather = [&](const tword* base, int b) {
          double g[RPL], s = 0.0;
          if constexpr (kTag) {
            tword w[2 * RPL];
            tag_load(w, [&](int k) { return tag_word(base, 64u * b + 8u * k); }, tag, fail);
#pragma unroll
            for (int q = 0; q < RPL; ++q) g[q] = tag_value<double>(w + 2 * q);
          } else {
#pragma unroll
            for (int q = 0; q < RPL; ++q) g[q] = cload(reinterpret_cast<const double*>(base + 8 * b + 2 * q));
          }
#pragma unroll
          for (int q = 0; q < RPL; ++q) s += g[q];
          return s;
        };
        s0 = s1 = 0.0;
#pragma unroll
        for (int h = 0; h < kScN; ++h) {
          const int b = sidx + h * (kGMax / kScN + 1);
          if (b < G && !pivot) s0 += gather(xb + ex.s0, b);
        }
        if (sidx < TR && !pivot) s1 = gather(xb + ex.s1, sidx);
        s0 = wsum(s0);
        s1 = wsum(s1);
        if (lane == 0) {
          red[0][swave] = s0;
          red[1][swave] = s1;
        }
      }
      if (pivot) {
        tword w[W];
        auto load = [&](int k) { return tag_word(xb + ex.al, 8u * k); };
        tag_load(w, load, tag, fail);
        piv[0] = tag_value<T>(w);
        piv[1] = y;
        piv[2] = a1;
      }
      __syncthreads();
      // v, w and the next u on the rows of the tile (the same values for a row
      // in every workgroup that has it)
      if (tid < TS || (offdiag && tid >= kKT && tid - kKT < TS)) {
        const bool isI = tid < TS;
        const int r = isI ? tid : tid - kKT;
        const Reflector f((double)piv[0], (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]),
                          (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]), (double)piv[1], (double)piv[2]);
        const T w1 = (T)f.w((double)piv[1], (double)piv[2], 1.0);
        T vr = T(0), wr = T(0), un = T(0);
        if (live) {
          const double vd = row == j + 1 ? 1.0 : f.c * (double)(isI ? uI[r] : uK[r]);
          vr = (T)vd;
          wr = (T)f.w((double)y, (double)a1, vd);
          un = a1 - (vr * w1 + wr);
          if (diag) {
            A[row + (unsigned)j * ld] = vr;
            if (row == j + 1) {
              a.d[j + 1] = un;
              a.e[j] = (T)f.beta;
              a.tau[j] = (T)f.tau;
            }
          }
        }
        if (row == j + 1) un = T(0);
        if (isI) {
          vw[sl][0][r] = vr;
          vw[sl][1][r] = wr;
          uI[r] = un;
        }
        if (diag || !isI) {
          vw[sl][2][r] = vr;
          vw[sl][3][r] = wr;
          uK[r] = un;
        }
      }
      __syncthreads();
      if constexpr (kDelta) {
        T vr[RPL], wr[RPL];
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
          vr[q] = vw[0][0][lane + q * kWave];
          wr[q] = vw[0][1][lane + q * kWave];
        }
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          const T vc = vw[0][2][cb + c], wc = vw[0][3][cb + c];
#pragma unroll
          for (int q = 0; q < RPL; ++q) dl[c][q] += vr[q] * wc + wr[q] * vc;
        }
      }
    }
    if constexpr (kDelta) {
#pragma unroll
      for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
          v[c][q] -= dl[c][q];
          dl[c][q] = T(0);
        }
    } else {
      constexpr int CC = 4;  // columns of the tile at a time
      static_assert(CW % CC == 0, "whole groups of columns");
#pragma unroll
      for (int c0 = 0; c0 < CW; c0 += CC) {
        T up[CC][RPL] = {};
#pragma clang loop unroll(disable)
        for (int t = 0; t < g1 - g0; ++t) {
          T vr[RPL], wr[RPL];
#pragma unroll
          for (int q = 0; q < RPL; ++q) {
            vr[q] = vw[t][0][lane + q * kWave];
            wr[q] = vw[t][1][lane + q * kWave];
          }
#pragma unroll
          for (int c = 0; c < CC; ++c) {
            const T vc = vw[t][2][cb + c0 + c], wc = vw[t][3][cb + c0 + c];
#pragma unroll
            for (int q = 0; q < RPL; ++q) up[c][q] += vr[q] * wc + wr[q] * vc;
          }
        }
#pragma unroll
        for (int c = 0; c < CC; ++c)
#pragma unroll
          for (int q = 0; q < RPL; ++q) {
            v[c0 + c][q] -= up[c][q];
            // here, not after the other groups' loops with up kept until then
            asm volatile("" : "+v"(v[c0 + c][q]));
          }
      }
    }
  }
  // the part of the tile that the next launch starts from
  const int jn = p + a.nc;
#pragma unroll
  for (int c = 0; c < CW; ++c)
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
      const int r = lane + q * kWave, k = cb + c;
      if (r < nI && k < nK && K0 + k >= jn && I0 + r >= K0 + k) A[I0 + r + (unsigned)(K0 + k) * ld] = v[c][q];
    }
}

// The last columns, once the trailing matrix A(p:n, p:n) has at most 64 Q
// rows: one workgroup per batch entry holds all of it in registers (wave w
// columns 4 Q w .., lane l rows l, l + 64, ..) and reduces ncol columns by the
// unblocked recurrence, with no exchange through memory and three workgroup
// barriers per column:
//   y = A u as one partial sum per wave and row;  ||u||^2, u^T y;
//   v = c (u - beta e1), w = tau A v - (tau^2 / 2)(v^T A v) v, and the next
//   column u' = A(:, j+1) - v w_{j+1} - w;  A -= v w^T + w v^T.
// 1.8 us per column on average from 256 rows (float), 1.4 from 64, where a
// launch with the exchange through memory took 7.2 us with one workgroup;
// bound by the instructions of the product and the update.  Larger trailing
// matrices do not fit the registers.  Reduced columns get their
// reflector; if columns remain, the lower triangle of the rest is written back.
constexpr int kTailThreads = 1024;
template <typename T, int Q>
__global__ __launch_bounds__(kTailThreads) void sytrd_tail_kernel(int n, int p, int ncol, T* A, T* d, T* e,
                                                              T* tau, int64_t sA, int64_t sD) {
  constexpr int NW = kTailThreads / kWave, R = kWave * Q, CW = R / NW;
  A += blockIdx.x * sA;
  d += blockIdx.x * sD;
  e += blockIdx.x * sD;
  tau += blockIdx.x * sD;
  const int M = n - p, tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), cb = wave * CW;
  __shared__ __attribute__((aligned(16))) T us[R], vs[R], ws[R];
  __shared__ T a1s[R], zred[NW][R], y1s;
  __shared__ double red[2][Q];
  T* Ap = A + p + (int64_t)p * n;
  T v[CW][Q];
#pragma unroll
  for (int c = 0; c < CW; ++c)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int row = lane + kWave * q, col = cb + c;
      v[c][q] = (row < M && col < M) ? Ap[max(row, col) + (int64_t)min(row, col) * n] : T(0);
    }
  // column jc into dst by its wave
  auto put_column = [&](int jc, T* dst) {
    if (jc < cb || jc >= cb + CW) return;
#pragma unroll
    for (int c = 0; c < CW; ++c)
      if (cb + c == jc) {
#pragma unroll
        for (int q = 0; q < Q; ++q) dst[lane + kWave * q] = v[c][q];
      }
  };
  put_column(0, us);
  put_column(1, a1s);
  __syncthreads();
  if (tid == 0) {
    d[p] = us[0];
    us[0] = T(0);
  }
  __syncthreads();
  for (int j = 0; j < ncol; ++j) {
    // partial y, one per wave with columns right of j
    if (cb + CW > j + 1) {
      T z[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) z[q] = T(0);
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const T uc = us[cb + c];
#pragma unroll
        for (int q = 0; q < Q; ++q) z[q] += v[c][q] * uc;
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) zred[wave][lane + kWave * q] = z[q];
    }
    __syncthreads();
    // rows: y, u^T y, ||u(2:)||^2
    T y = T(0), ur = T(0), alpha = T(0);
    if (tid < R) {
      const int wlo = (j + 1) / CW;
#pragma unroll
      for (int w = 0; w < NW; ++w) y += w >= wlo ? zred[w][tid] : T(0);
      ur = us[tid];
      alpha = us[j + 1];
      if (tid == j + 1) y1s = y;
      const double s0 = wsum((double)ur * (double)y);
      const double s1 = wsum(tid >= j + 2 ? (double)ur * (double)ur : 0.0);
      if (lane == 0) {
        red[0][wave] = s0;
        red[1][wave] = s1;
      }
    }
    __syncthreads();
    if (tid < R) {
      double uAu = 0.0, sig = 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        uAu += red[0][q];
        sig += red[1][q];
      }
      const double al = (double)alpha, y1 = (double)y1s, a11 = (double)a1s[j + 1];
      const Reflector f(al, sig, uAu, y1, a11);
      const T w1 = (T)f.w(y1, a11, 1.0);
      T vr = T(0), wr = T(0), un = T(0);
      if (tid >= j + 1) {
        const T ar = a1s[tid];
        const double vd = tid == j + 1 ? 1.0 : f.c * (double)ur;
        vr = (T)vd;
        wr = (T)f.w((double)y, (double)ar, vd);
        un = ar - (vr * w1 + wr);
        if (tid < M) Ap[tid + (int64_t)j * n] = vr;
      }
      vs[tid] = vr;
      ws[tid] = wr;
      us[tid] = tid > j + 1 ? un : T(0);
      if (tid == j + 1) {
        d[p + j + 1] = un;
        e[p + j] = (T)f.beta;
        tau[p + j] = (T)f.tau;
      }
    }
    __syncthreads();
    if (cb + CW > j + 1) {
      T vr[Q], wr[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        vr[q] = vs[lane + kWave * q];
        wr[q] = ws[lane + kWave * q];
      }
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const T vc = vs[cb + c], wc = ws[cb + c];
#pragma unroll
        for (int q = 0; q < Q; ++q) v[c][q] -= vr[q] * wc + wr[q] * vc;
      }
    }
    put_column(j + 2, a1s);
  }
  if (ncol < M - 1) {
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int row = lane + kWave * q, col = cb + c;
        if (col >= ncol && row >= col && row < M) Ap[row + (int64_t)col * n] = v[c][q];
      }
  }
}

// Rows of the trailing matrix that the tail takes over: the registers hold
// 64 values per thread in float and 36 in double.
template <typename T>
constexpr int kTailRows = sizeof(T) == 4 ? 256 : 192;

template <typename T>
void launch_tail(hipStream_t st, int n, int p, int batch, T* A, int64_t sA, T* d, T* e, T* tau, int64_t sD) {
  while (p < n - 1) {
    const int M = n - p, q = (int)ceil_div(M, kWave);
    // down to the next smaller register tile
    const int ncol = q == 1 ? M - 1 : M - kWave * (q - 1);
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(batch), dim3(kTailThreads), 0, st, n, p, ncol, A, d, e, tau, sA, sD);
      MSQRT_LAUNCH_CHECK();
    };
    const int tok = prof_begin(st);
    if (q == 1) go(sytrd_tail_kernel<T, 1>);
    else if (q == 2) go(sytrd_tail_kernel<T, 2>);
    else if (q == 3) go(sytrd_tail_kernel<T, 3>);
    else if constexpr (sizeof(T) == 4) go(sytrd_tail_kernel<T, 4>);
    if (tok >= 0)
      prof_end(tok, st, sizeof(T) == 4 ? "sytrd_tail_f32" : "sytrd_tail_f64",
               4.0 * (double)M * M * ncol * batch, 8.0 * sizeof(T) * (double)M * M * batch / 8.0);
    p += ncol;
  }
}

// Largest co-resident grid of one panel kernel.
template <typename T, int RPL>
int panel_resident() {
  static const int r = [] {
    int per_cu = 0, ncu = 0, dev = 0;
    MSQRT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, (const void*)sytrd_panel_kernel<T, RPL>, (Tile<T, RPL>::NT), 0));
    MSQRT_HIP(hipGetDevice(&dev));
    MSQRT_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    return std::max(1, std::min(per_cu, 1)) * std::max(1, ncu);  // one workgroup per CU
  }();
  return r;
}

// One panel launch: columns p .. p + nc - 1 with tiles of 64 rpl rows, TR per
// dimension, `chunk` batch entries at a time.
struct PanelLaunch {
  int p, nc, rpl, TR, chunk;
};

// The launches that leave kTailRows rows; res[rpl - 1]: co-resident workgroups.
// Tile of 64 rpl rows: a small tile has less work per column (n = 1000: 4.15 ms
// with 64 rows, 4.4 with 128, 5.1 with 192, 5.5 with 256) but needs more
// workgroups; a batch that is not co-resident takes several launches, each as
// long as one (64 x 512: 2.3 ms with 256 rows in one launch, 2.8 with 192 in two,
// 4.1 with 128 in three, all with the barrier; with tags the 64-row tiles took
// 3.4 ms at n = 1000).
template <typename T>
std::vector<PanelLaunch> panel_launches(int n, int batch, const int (&res)[4]) {
  std::vector<PanelLaunch> plan;
  for (int p = 0; n - p > kTailRows<T>; p += plan.back().nc) {
    const int m = n - p;
    PanelLaunch best{p, std::min(kLaunchCols, m - kTailRows<T>), 0, 0, 0};
    double cost = 0.0;
    for (int rpl = 1; rpl <= 4; ++rpl) {
      const int tr = (int)ceil_div(m, kWave * rpl), g = tr * (tr + 1) / 2;
      if (tr > kTRMax || g > res[rpl - 1]) continue;
      const int ch = std::min(batch, res[rpl - 1] / g);
      // (256-row tiles of doubles spill: for the one order that needs them)
      const double c = (double)ceil_div(batch, ch) * (5.0 + 0.25 * rpl * rpl) * (rpl == 4 && sizeof(T) == 8 ? 8.0 : 1.0);
      if (best.rpl == 0 || c < cost) {
        best = {p, best.nc, rpl, tr, ch};
        cost = c;
      }
    }
    if (best.rpl == 0) throw Error{MSQRT_ERR_UNSUPPORTED, "tridiagonal reduction: the device holds too few workgroups"};
    plan.push_back(best);
  }
  return plan;
}

// Words that one batch entry's launches exchange through: two buffers of the
// largest layout among them.
template <typename T>
int64_t exchange_words(int n, const std::vector<PanelLaunch>& plan) {
  int64_t size = 0;
  for (const PanelLaunch& l : plan) size = std::max(size, Exchange<T>(n, l.TR).size);
  return 2 * size;
}

template <typename T>
__global__ void copy_diag(const T* A, T* d, int64_t sA, int64_t sD) {
  if (threadIdx.x == 0) d[blockIdx.x * sD] = A[blockIdx.x * sA];
}

}  // namespace

int sytrd_max_n() { return kMaxN; }
static_assert((int64_t)kMaxN * kMaxN < (int64_t(1) << 31), "the kernels' 32-bit offsets cover an n x n matrix");
static_assert(kMaxN < (int)kTagSteps - 1, "one tag per column");
unsigned sytrd_tag(int column) { return step_tag((unsigned)column); }

template <typename T>
void sytrd_batched(hipStream_t st, int n, int batch, T* A, int64_t sA, T* d, T* e, T* tau,
                   int64_t sD, SytrdWork& w) {
  if (n <= 0 || batch <= 0) return;
  if (n == 1) {
    hipLaunchKernelGGL(copy_diag<T>, dim3(batch), 64, 0, st, (const T*)A, d, sA, sD);
    MSQRT_LAUNCH_CHECK();
    return;
  }
  if (n > sytrd_max_n())
    throw Error{MSQRT_ERR_UNSUPPORTED, "tridiagonal reduction supports n <= 4225 in this build"};
  w.nbar = n > kTailRows<T> ? batch : 0;  // entries that exchange words
  if (w.nbar == 0) {
    launch_tail<T>(st, n, 0, batch, A, sA, d, e, tau, sD);
    return;
  }
  const int res[4] = {panel_resident<T, 1>(), panel_resident<T, 2>(), panel_resident<T, 3>(), panel_resident<T, 4>()};
  const std::vector<PanelLaunch> plan = panel_launches<T>(n, batch, res);
  const int64_t sX = exchange_words<T>(n, plan);
  tword* x = w.x.ensure<tword>(sX * batch);
  unsigned* bar = w.bar.ensure<unsigned>((int64_t)kBarWords * batch);
  // no word carries a tag yet
  MSQRT_HIP(hipMemsetAsync(x, 0, sizeof(tword) * (size_t)(sX * batch), st));
  MSQRT_HIP(hipMemsetAsync(bar, 0, sizeof(unsigned) * (size_t)kBarWords * batch, st));
  BarrierBase bar_base{};
  for (const PanelLaunch& l : plan) {
    const int p = l.p, m = n - p, nc = l.nc, best = l.rpl, TR = l.TR, chunk = l.chunk;
    const int G = TR * (TR + 1) / 2, ts = (int)ceil_div(m, TR);
    const int tok = prof_begin(st);
    for (int b0 = 0; b0 < batch; b0 += chunk) {
      PanelArgs<T> pa{n,  p,  nc, TR, ts, A + b0 * sA, d + b0 * sD, e + b0 * sD, tau + b0 * sD,
                      x + b0 * sX, bar + (int64_t)b0 * kBarWords, bar_base, sA, sD, sX};
      void* args[] = {&pa};
      const int nt = best == 1 ? Tile<T, 1>::NT : best == 2 ? Tile<T, 2>::NT : best == 3 ? Tile<T, 3>::NT : Tile<T, 4>::NT;
      const void* kern = best == 1 ? (const void*)sytrd_panel_kernel<T, 1>
                         : best == 2 ? (const void*)sytrd_panel_kernel<T, 2>
                         : best == 3 ? (const void*)sytrd_panel_kernel<T, 3>
                                     : (const void*)sytrd_panel_kernel<T, 4>;
      MSQRT_HIP(hipLaunchCooperativeKernel(kern, dim3(G, std::min(chunk, batch - b0)), dim3(nt), args, 0, st));
    }
    const bool tag = best == 1 ? Tile<T, 1>::kTag : best == 2 ? Tile<T, 2>::kTag : best == 3 ? Tile<T, 3>::kTag : Tile<T, 4>::kTag;
    if (!tag) {
      bar_base.gen += (unsigned)nc;
      bar_base.top += (unsigned)std::min(G, 8) * (unsigned)nc;
      if (G > 8)  // with fewer workgroups the barrier skips the group counters
        for (int g = 0; g < 8; ++g) bar_base.sub[g] += (unsigned)(G / 8 + (g < G % 8 ? 1 : 0)) * (unsigned)nc;
    }
    if (tok >= 0) {
      // what the launch has to move: the lower triangle of the trailing matrix
      // into registers, the rest of it back, and the reflectors
      const double r = m - nc, bytes = (0.5 * m * (m + 1.0) + 0.5 * r * (r + 1.0) + (double)nc * m) * sizeof(T);
      prof_end(tok, st, sizeof(T) == 4 ? "sytrd_panel_f32" : "sytrd_panel_f64",
               4.0 * (double)m * m * nc * batch, bytes * batch);
    }
  }
  launch_tail<T>(st, n, plan.back().p + plan.back().nc, batch, A, sA, d, e, tau, sD);
}

template <typename T>
int64_t sytrd_exchange_bytes(int n, int batch, int cus) {
  const int res[4] = {cus, cus, cus, cus};
  return (int64_t)sizeof(tword) * exchange_words<T>(n, panel_launches<T>(n, batch, res));
}
template int64_t sytrd_exchange_bytes<float>(int, int, int);
template int64_t sytrd_exchange_bytes<double>(int, int, int);

template <typename T>
void sytrd(hipStream_t st, int n, T* A, T* d, T* e, T* tau, SytrdWork& w) {
  sytrd_batched<T>(st, n, 1, A, (int64_t)n * n, d, e, tau, 0, w);
}

bool sytrd_failed(SytrdWork& w) {
  if (!w.bar.p || w.nbar <= 0) return false;
  std::vector<unsigned> flags((size_t)kBarWords * w.nbar);
  MSQRT_HIP(hipMemcpy(flags.data(), w.bar.p, sizeof(unsigned) * flags.size(), hipMemcpyDeviceToHost));
  for (int b = 0; b < w.nbar; ++b)
    if (flags[(size_t)b * kBarWords + kBarFail]) return true;
  return false;
}

template void sytrd<float>(hipStream_t, int, float*, float*, float*, float*, SytrdWork&);
template void sytrd<double>(hipStream_t, int, double*, double*, double*, double*, SytrdWork&);
template void sytrd_batched<float>(hipStream_t, int, int, float*, int64_t, float*, float*, float*,
                                   int64_t, SytrdWork&);
template void sytrd_batched<double>(hipStream_t, int, int, double*, int64_t, double*, double*,
                                    double*, int64_t, SytrdWork&);

}  // namespace msqrt
