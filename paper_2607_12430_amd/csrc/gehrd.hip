// Blocked Householder reduction to upper Hessenberg form, real or complex,
// for the Schur factorisation of the general path (Alg. 2, first line: the
// Schur decomposition starts from a Hessenberg reduction).
//
// Panels of up to kNb columns, one cooperative launch each.  A workgroup owns
// a block of rows of A, V and Y for the whole panel.  Column c = p + i is
// brought up to date from Y = A V T, V and T,
//   w = A(:, c) - Y V(c, :)^*,   w <- w - V T^* (V^* w)  (rows > p),
// its reflector H_c = I - tau v v^* is generated, y = A v is formed (A = the
// matrix at the start of the panel) and Y's next column is
// tau (y - Y (V^* v)).  Only V^* w, V^* v, the norm of w and w itself cross
// workgroups, so a column costs two grid barriers; y needs none, because a
// workgroup has whole rows of A, which it keeps in registers.  (One workgroup
// per column and a separate matrix-vector launch took 33 us per column at
// n = 2048, 18 us at n = 333, most of it one CU reading V and Y back.)
// Matrices of at most kSolo rows take one workgroup and no grid barrier.
//
// After the panel, with W = V^* A(:, q:) - (V^* Y) V(q:, :)^*,
//   A(:, q:) -= Y V(q:, :)^* + V (T^* W)
// as a split-K product for V^* [A Y], one small launch for T^* W and one
// MFMA GEMM of inner dimension 2 kNb (4 kNb for complex).  Q1 = H_0 H_1 ...
// is formed by applying the block reflectors to the identity, last block
// first, with the same three launches.
#include <algorithm>

#include "gemm.hpp"
#include "gridsync.hpp"
#include "kernels.hpp"
#include "schur.hpp"

namespace msqrt {

namespace {

constexpr int kNb = 32;
constexpr int kThreads = kSyncThreads;
constexpr int kMaxG = 256;
constexpr int kSolo = 128;
constexpr int kLd = kNb + 1;  // LDS row stride of the kNb-column arrays
constexpr size_t kLdsMax = 150 * 1024;
constexpr int kMaxBy = 8;  // workgroups (of four K-chunks) per 32 columns of a V^* product
constexpr int kPad = 8 * (kThreads / 16);  // zeros behind the exchanged column in LDS: one group of 8 per lane

// Squared norm of a column (of a matrix scaled to about 1) below which it counts
// as reduced: its squares lose digits or underflow, and v would not be the
// reflector of tau.  Its norm is far below the rounding of the reduction.
template <typename T>
constexpr T kTinyNorm2 = sizeof(T) == 4 ? T(1e-30) : T(1e-280);

// Element arithmetic shared by the real and the complex reduction.
template <typename T>
struct HReal {
  using E = T;
  static constexpr int P = 1;  // planes
  __host__ __device__ static E zero() { return T(0); }
  __device__ static E load(const T* p, int64_t) { return p[0]; }
  __device__ static void store(T* p, int64_t, E v) { p[0] = v; }
  __device__ static E cl(const E* p) { return cload(p); }
  __device__ static void cs(E* p, E v) { cstore(p, v); }
  __device__ static E add(E a, E b) { return a + b; }
  __device__ static E sub(E a, E b) { return a - b; }
  __device__ static E mul(E a, E b) { return a * b; }
  __device__ static E mulc(E a, E b) { return a * b; }  // conj(a) b
  __device__ static E conj(E a) { return a; }
  __device__ static T abs2(E a) { return a * a; }
  __device__ static E real(T v) { return v; }
  __device__ static T re(E a) { return a; }
  __device__ static E sum16(E a) { return rsum16(a); }
  // tau, scal with v = scal (w - beta e_1), for alpha = w_1, s2 = |w_2..|^2
  __device__ static void reflector(E alpha, T s2, T& beta, E& tau, E& scal) {
    beta = alpha;
    tau = scal = T(0);
    const T n2 = alpha * alpha + s2;
    if (s2 == T(0) || n2 < kTinyNorm2<T>) return;
    beta = -copysign(sqrt(n2), alpha);
    tau = (beta - alpha) / beta;
    scal = T(1) / (alpha - beta);
  }
  // entry c+1 of the reduced column
  __device__ static E corner(E, T beta) { return beta; }
};
template <typename T>
struct HCplx {
  using E = cx<T>;
  static constexpr int P = 2;
  __host__ __device__ static E zero() { return {T(0), T(0)}; }
  __device__ static E load(const T* p, int64_t im) { return {p[0], p[im]}; }
  __device__ static void store(T* p, int64_t im, E v) {
    p[0] = v.r;
    p[im] = v.i;
  }
  __device__ static E cl(const E* p) { return {cload(&p->r), cload(&p->i)}; }
  __device__ static void cs(E* p, E v) {
    cstore(&p->r, v.r);
    cstore(&p->i, v.i);
  }
  __device__ static E add(E a, E b) { return cadd(a, b); }
  __device__ static E sub(E a, E b) { return csub(a, b); }
  __device__ static E mul(E a, E b) { return cmul(a, b); }
  __device__ static E mulc(E a, E b) { return cmulc(a, b); }
  __device__ static E conj(E a) { return cconj(a); }
  __device__ static T abs2(E a) { return cabs2(a); }
  __device__ static E real(T v) { return {v, T(0)}; }
  __device__ static T re(E a) { return a.r; }
  __device__ static E sum16(E a) { return {rsum16(a.r), rsum16(a.i)}; }
  __device__ static void reflector(E alpha, T s2, T& beta, E& tau, E& scal) {
    beta = alpha.r;
    tau = scal = zero();
    const T n2 = alpha.r * alpha.r + alpha.i * alpha.i + s2;
    if ((s2 == T(0) && alpha.i == T(0)) || n2 < kTinyNorm2<T>) return;
    beta = -copysign(sqrt(n2), alpha.r);
    tau = {(beta - alpha.r) / beta, -alpha.i / beta};
    scal = cdiv(cx<T>{T(1), T(0)}, csub(alpha, cx<T>{beta, T(0)}));
  }
  __device__ static E corner(E, T beta) { return {beta, T(0)}; }
};

template <typename T, class F>
struct PanelArgs {
  int n, p, nbp;
  int rbp, G;    // rows per workgroup (a power of two), workgroups
  int nbw;       // columns of a full panel
  int wf_lds;    // the exchanged column fits LDS
  T* H;          // ld P n, imaginary plane n rows below
  T* V;          // P planes of n x kNb, ld n: this panel's reflectors
  T* YV;         // P times [Y plane, V plane], each n x kNb, ld n
  T* Tp;         // P planes of kNb x kNb
  typename F::E* wbuf;  // the updated column
  typename F::E* up;    // G x kNb partial sums of V^* w
  typename F::E* sp;    // G x kNb partial sums of V^* w_tail; slot kNb - 1: |w_tail|^2
  unsigned* bar;
  BarrierBase bar_base;
};

template <class F>
size_t panel_lds(int rbp, int n, bool wf, int nbw = kNb) {
  const size_t e = (size_t)3 * rbp * (nbw + 1) + 2 * kNb * kLd + kThreads + kNb * kLd + rbp + 4 * kNb +
                   (wf ? (size_t)n + kPad : 0);
  return e * sizeof(typename F::E);
}

// KREG: elements of A's rows held in registers per thread (the rest is read
// from L2 at every column).  kW: columns of a panel, 0 = a.nbw of them (the
// large blocks of rows of the largest matrices, where LDS has no room for kNb).
template <typename T, class F, int KREG, int kW>
__global__ __launch_bounds__(kThreads) void hess_panel_kernel(PanelArgs<T, F> a) {
  using E = typename F::E;
  const int n = a.n, p = a.p, rbp = a.rbp, G = a.G;
  const int lv = (kW ? kW : a.nbw) + 1;  // LDS row stride of V, Y and A's columns
  const int64_t ldh = (int64_t)F::P * n;
  const int blk = blockIdx.x, r0 = blk * rbp;
  const int t = threadIdx.x, g16 = t >> 4, l = t & 15;
  const bool solo = G == 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  E* Vl = reinterpret_cast<E*>(smem);  // [r][k]
  E* Yl = Vl + rbp * lv;
  E* Ap = Yl + rbp * lv;              // the panel's columns of A, own rows
  E* Tl = Ap + rbp * lv;              // [row][column]
  E* PV = Tl + kNb * kLd;              // V(p + 1 + q, k)
  E* red = PV + kNb * kLd;
  E* wl = red + kThreads + kNb * kLd;  // own rows of the column
  E* us = wl + rbp;
  E* zs = us + kNb;
  E* vt = zs + kNb;                    // V^* v
  E* al = vt + kNb;                    // alpha
  E* wf = al + kNb;                    // rows p + 1 .. of the exchanged column
  unsigned sub_base = 0;
#pragma unroll
  for (int g = 0; g < 8; ++g)
    if (g == (blk & 7)) sub_base = a.bar_base.sub[g];
  int nbar = 0;

  for (int x = t; x < rbp * lv; x += kThreads) {
    const int r = x / lv, k = x % lv;
    Vl[x] = Yl[x] = F::zero();
    Ap[x] = (r0 + r < n && k < a.nbp) ? F::load(a.H + r0 + r + (int64_t)(p + k) * ldh, n) : F::zero();
  }
  for (int x = t; x < kNb * kLd; x += kThreads) Tl[x] = PV[x] = F::zero();
  if (a.wf_lds)
    for (int x = t; x < kPad; x += kThreads) wf[n + x] = F::zero();

  // rows of A right of column p: thread (gr, cg) holds the elements of row gr
  // in columns p + 1 + cg + CG k
  const int gr = t & (rbp - 1), cg = t / rbp, CG = kThreads / rbp;
  const int nk = (n - p - 1 + CG - 1) / CG;
  const int grow = min(r0 + gr, n - 1);
  E tile[KREG];
#pragma unroll
  for (int k = 0; k < KREG; ++k) {
    const int c = p + 1 + cg + CG * k;
    tile[k] = c < n ? F::load(a.H + grow + (int64_t)c * ldh, n) : F::zero();
  }
  __syncthreads();

  // sum over the workgroups of their kNb partial values, into out[]
  auto gather = [&](const E* part, E* out) {
    const int k = t & (kNb - 1), gg = t / kNb;
    E v[kMaxG / kNb];
#pragma unroll
    for (int m = 0; m < kMaxG / kNb; ++m) {
      const int g = gg + kNb * m;
      v[m] = g < G ? F::cl(part + g * kNb + k) : F::zero();
    }
    E s = v[0];
#pragma unroll
    for (int m = 1; m < kMaxG / kNb; ++m) s = F::add(s, v[m]);
    red[gg * kLd + k] = s;
    __syncthreads();
    if (t < kNb * 16) {
      const E x = F::sum16(F::add(red[l * kLd + g16], red[(l + 16) * kLd + g16]));
      if (l == 0) out[g16] = x;
    }
  };

  for (int i = 0; i < a.nbp; ++i) {
    const int c = p + i;
    // w = A(:, c) - Y V(c, :)^*
    for (int r = g16; r < rbp; r += kThreads / 16) {
      E s = F::zero();
      for (int k = l; k < i; k += 16) s = F::add(s, F::mulc(PV[(i - 1) * kLd + k], Yl[r * lv + k]));
      s = F::sum16(s);
      if (l == 0) wl[r] = F::sub(Ap[r * lv + i], s);
    }
    __syncthreads();
    if (i > 0) {
      // w <- w - V T^* (V^* w); V is zero in the rows <= p
      if (t < kNb * 16) {
        E s = F::zero();
        if (g16 < i)
          for (int r = l; r < rbp; r += 16) s = F::add(s, F::mulc(Vl[r * lv + g16], wl[r]));
        s = F::sum16(s);
        if (l == 0) {
          if (solo) us[g16] = s;
          else F::cs(a.up + blk * kNb + g16, s);
        }
      }
      if (solo) {
        __syncthreads();
      } else {
        grid_barrier(a.bar, a.bar_base, sub_base, blk, G, ++nbar);
        gather(a.up, us);
        __syncthreads();
      }
      if (t < kNb * 16) {
        E s = F::zero();
        for (int j = l; j < i; j += 16)
          if (j <= g16) s = F::add(s, F::mulc(Tl[j * kLd + g16], us[j]));
        s = F::sum16(s);
        if (l == 0) zs[g16] = s;
      }
      __syncthreads();
      for (int r = g16; r < rbp; r += kThreads / 16) {
        E s = F::zero();
        for (int k = l; k < i; k += 16) s = F::add(s, F::mul(Vl[r * lv + k], zs[k]));
        s = F::sum16(s);
        if (l == 0) wl[r] = F::sub(wl[r], s);
      }
      __syncthreads();
    }
    // partial V^* w and |w|^2 over the rows >= c + 2; the rows >= c + 1 of w
    if (t < kNb * 16) {
      E s = F::zero();
      for (int r = l; r < rbp; r += 16)
        if (r0 + r >= c + 2) {
          if (g16 < i) s = F::add(s, F::mulc(Vl[r * lv + g16], wl[r]));
          else if (g16 == kNb - 1) s = F::add(s, F::real(F::abs2(wl[r])));
        }
      s = F::sum16(s);
      if (l == 0) {
        if (solo) us[g16] = s;
        else F::cs(a.sp + blk * kNb + g16, s);
      }
    } else if (t - kNb * 16 < rbp) {
      const int r = t - kNb * 16, row = r0 + r;
      if (row < n && row > p) {
        const E w = row > c ? wl[r] : F::zero();
        if (!solo) F::cs(a.wbuf + row, w);
        else wf[row] = w;
        if (solo && row == c + 1) al[0] = w;
      }
    }
    if (solo) {
      __syncthreads();
    } else {
      grid_barrier(a.bar, a.bar_base, sub_base, blk, G, ++nbar);
      if (a.wf_lds) {
        for (int row = p + 1 + t; row < n; row += kThreads) {
          const E w = F::cl(a.wbuf + row);
          wf[row] = w;
          if (row == c + 1) al[0] = w;
        }
      } else if (t == 0) {
        al[0] = F::cl(a.wbuf + c + 1);
      }
      gather(a.sp, us);
      __syncthreads();
    }
    // the reflector v = scal (w - beta e_{c+1}), the same in every workgroup
    const E alpha = al[0];
    T beta;
    E tau, scal;
    F::reflector(alpha, F::re(us[kNb - 1]), beta, tau, scal);
    const E head = F::sub(alpha, F::real(beta));
    if (t < kNb) {
      const int row = p + 1 + t;
      E v = F::zero();
      if (row == c + 1) v = F::real(T(1));
      else if (row > c + 1 && row < n) v = F::mul(scal, a.wf_lds ? wf[row] : F::cl(a.wbuf + row));
      PV[t * kLd + i] = v;
    } else if (t >= kWave && t < kWave + kNb) {
      const int k = t - kWave;
      if (k < i) vt[k] = F::add(F::conj(PV[i * kLd + k]), F::mul(scal, us[k]));
    } else if (t >= kNb * 16 && t - kNb * 16 < rbp) {
      const int r = t - kNb * 16, row = r0 + r;
      if (row < n) {
        E v = F::zero();
        if (row == c + 1) v = F::real(T(1));
        else if (row > c + 1) v = F::mul(scal, wl[r]);
        Vl[r * lv + i] = v;
        F::store(a.H + row + (int64_t)c * ldh, n,
                 row <= c ? wl[r] : (row == c + 1 ? F::corner(alpha, beta) : F::zero()));
      }
    }
    if (t == 2 * kWave && a.wf_lds) wf[c + 1] = head;
    __syncthreads();
    // y = A v = scal (A w'), w' = w with alpha - beta in row c + 1
    {
      E s = F::zero();
      if (a.wf_lds) {
        const E* wp = wf + p + 1 + cg;
#pragma unroll
        for (int k8 = 0; k8 < KREG; k8 += 8)
          if (k8 < nk) {
#pragma unroll
            for (int k = k8; k < k8 + 8; ++k) s = F::add(s, F::mul(tile[k], wp[CG * k]));
          }
        for (int k = KREG; k < nk; ++k) {
          const int col = p + 1 + cg + CG * k;
          if (col < n) s = F::add(s, F::mul(F::load(a.H + grow + (int64_t)col * ldh, n), wf[col]));
        }
      } else {
        for (int k = 0; k < nk; ++k) {
          const int col = p + 1 + cg + CG * k;
          if (col < n)
            s = F::add(s, F::mul(F::load(a.H + grow + (int64_t)col * ldh, n),
                                 col == c + 1 ? head : F::cl(a.wbuf + col)));
        }
      }
      red[t] = s;
    }
    // T(:i, i) = -tau T(:i, :i) (V^* v)
    if (t < kNb * 16) {
      E s = F::zero();
      for (int k = l; k < i; k += 16)
        if (k >= g16) s = F::add(s, F::mul(Tl[g16 * kLd + k], vt[k]));
      s = F::sum16(s);
      if (l == 0 && g16 < i) Tl[g16 * kLd + i] = F::sub(F::zero(), F::mul(tau, s));
      if (l == 0 && g16 == i) Tl[g16 * kLd + i] = tau;
    }
    __syncthreads();
    // Y(:, i) = tau (y - Y (V^* v))
    for (int r = g16; r < rbp; r += kThreads / 16) {
      E s = F::zero();
      for (int q = l; q < CG; q += 16) s = F::add(s, red[q * rbp + r]);
      s = F::mul(scal, s);
      for (int k = l; k < i; k += 16) s = F::sub(s, F::mul(Yl[r * lv + k], vt[k]));
      s = F::sum16(s);
      if (l == 0) Yl[r * lv + i] = r0 + r < n ? F::mul(tau, s) : F::zero();
    }
    __syncthreads();
  }

  const int64_t pl = (int64_t)n * kNb;
  for (int x = t; x < rbp * kNb; x += kThreads) {
    const int r = x % rbp, k = x / rbp, row = r0 + r;
    if (row >= n) continue;
    const E v = k < lv - 1 ? Vl[r * lv + k] : F::zero(), y = k < lv - 1 ? Yl[r * lv + k] : F::zero();
    F::store(a.V + row + (int64_t)k * n, pl, v);
    F::store(a.YV + row + (int64_t)k * n, 2 * pl, y);
    F::store(a.YV + pl + row + (int64_t)k * n, 2 * pl, v);
  }
  if (blk == 0)
    for (int x = t; x < kNb * kNb; x += kThreads) F::store(a.Tp + x, kNb * kNb, Tl[(x % kNb) * kLd + x / kNb]);
}

// Partial products of V(r0 : r0+K, 0:kNb)^* B(r0 : r0+K, :), B = N columns of
// B followed by N2 columns of B2.  One wave per 32 columns and K-chunk, both
// operands read straight from memory (both are k-contiguous, a lane takes
// four k at a time); chunk s of column j: Wp[((s P + plane) (N + N2) + j) kNb + m].
template <typename T, class F>
__global__ __launch_bounds__(256) void vta_kernel(int K, int chunk, int N, int N2, const T* V, int64_t ldv,
                                                  int64_t vim, const T* B, int64_t ldb, int64_t bim,
                                                  const T* B2, int64_t ldb2, int64_t b2im, T* Wp) {
  using M = Mfma<T>;
  constexpr int P = F::P, TM = M::TM, NB = 32 / TM, KG = kWave / TM * 4;
  const int lane = threadIdx.x % kWave, s = blockIdx.y * 4 + threadIdx.x / kWave;
  const int k0 = s * chunk, k1 = min(K, k0 + chunk), NN = N + N2;
  const int mn = lane % TM, kk = lane / TM;
  const T *vp[NB], *bp[NB];
  int64_t bi[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    vp[b] = V + (int64_t)(b * TM + mn) * ldv;
    const int j = min(32 * (int)blockIdx.x + b * TM + mn, NN - 1);
    bp[b] = j < N ? B + j * ldb : B2 + (j - N) * ldb2;
    bi[b] = j < N ? bim : b2im;
  }
  typename M::acc_t acc[P][NB][NB];
#pragma unroll
  for (int q = 0; q < P; ++q)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int c = 0; c < NB; ++c) acc[q][b][c] = typename M::acc_t{};
  for (int k = k0 + 4 * kk; k - 4 * kk < k1; k += KG) {
    T vf[P][NB][4], bf[P][NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = k + e < k1;
        const int o = in ? k + e : k0;
        vf[0][b][e] = in ? vp[b][o] : T(0);
        bf[0][b][e] = in ? bp[b][o] : T(0);
        if constexpr (P == 2) {
          vf[1][b][e] = in ? vp[b][o + vim] : T(0);
          bf[1][b][e] = in ? bp[b][o + bi[b]] : T(0);
        }
      }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int c = 0; c < NB; ++c) {
          acc[0][b][c] = M::mma(vf[0][b][e], bf[0][c][e], acc[0][b][c]);
          if constexpr (P == 2) {
            // conj(V) B
            acc[0][b][c] = M::mma(vf[1][b][e], bf[1][c][e], acc[0][b][c]);
            acc[1][b][c] = M::mma(vf[0][b][e], bf[1][c][e], acc[1][b][c]);
            acc[1][b][c] = M::mma(-vf[1][b][e], bf[0][c][e], acc[1][b][c]);
          }
        }
  }
#pragma unroll
  for (int q = 0; q < P; ++q)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int r = 0; r < M::NACC; ++r) {
          const int j = 32 * blockIdx.x + c * TM + M::c_col(lane, r);
          if (j < NN) Wp[((int64_t)(s * P + q) * NN + j) * kNb + b * TM + M::c_row(lane, r)] = acc[q][b][c][r];
        }
}

// Per 32 columns: W = sum of the partials; kHess: W -= (V^* Y) V2^* (V2 =
// V(q:, :), the Y columns follow the N others in the partials) and W2 =
// T^* W; else W2 = T W.  The second operand of the update GEMMs is written as
// X = W2^* (N x kNb, ld N): plane order per output plane such that
// C -= [Y V] B^T (kHess) or V B^T; for complex, Re C from B = [Re, Im] and
// Im C from B = [-Im, Re], each with the planes of V2 before those of X.
template <typename T, class F, bool kHess>
__global__ __launch_bounds__(256) void w2_kernel(int splits, int N, const T* Wp, const T* Tp, const T* V2,
                                                 int64_t ldv, int64_t vim, T* Bo) {
  using E = typename F::E;
  constexpr int P = F::P;
  __shared__ E W[kNb * kLd], Ml[kHess ? kNb * kLd : 1], Tl[kNb * kLd], Vl[kHess ? kNb * kLd : 1];
  const int t = threadIdx.x, j0 = 32 * blockIdx.x, NN = kHess ? N + kNb : N;
  auto total = [&](int j, int m) {
    // splits is a multiple of 4; eight loads in flight
    E s = F::zero();
    const T* w = Wp + (int64_t)j * kNb + m;
    const int64_t im = (int64_t)NN * kNb;
    for (int q = 0; q < splits; q += 8) {
      E v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = q + e < splits ? F::load(w + (q + e) * P * im, im) : F::zero();
#pragma unroll
      for (int e = 0; e < 8; ++e) s = F::add(s, v[e]);
    }
    return s;
  };
  for (int x = t; x < kNb * kNb; x += 256) {
    const int m = x % kNb, j = x / kNb;
    W[m * kLd + j] = j0 + j < N ? total(j0 + j, m) : F::zero();
    Tl[m * kLd + j] = F::load(Tp + x, kNb * kNb);
    if constexpr (kHess) {
      Ml[m * kLd + j] = total(N + j, m);
      Vl[m * kLd + j] = j0 + m < N ? F::load(V2 + j0 + m + j * ldv, vim) : F::zero();  // [row][k]
    }
  }
  __syncthreads();
  if constexpr (kHess) {
    E w[kNb * kNb / 256];
#pragma unroll
    for (int e = 0; e < kNb * kNb / 256; ++e) {
      const int x = t + 256 * e, m = x % kNb, j = x / kNb;
      E s = W[m * kLd + j];
      for (int k = 0; k < kNb; ++k) s = F::sub(s, F::mulc(Vl[j * kLd + k], Ml[m * kLd + k]));
      w[e] = s;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kNb * kNb / 256; ++e) {
      const int x = t + 256 * e;
      W[x % kNb * kLd + x / kNb] = w[e];
    }
    __syncthreads();
  }
  const int64_t pl = (int64_t)N * kNb;
  constexpr int kPl = kHess ? 2 : 1;  // planes of B per plane of the factors
  for (int x = t; x < kNb * kNb; x += 256) {
    const int j = x % kNb, m = x / kNb;
    if (j0 + j >= N) continue;
    E s = F::zero();
    if (kHess)
      for (int k = 0; k <= m; ++k) s = F::add(s, F::mulc(Tl[k * kLd + m], W[k * kLd + j]));
    else
      for (int k = m; k < kNb; ++k) s = F::add(s, F::mul(Tl[m * kLd + k], W[k * kLd + j]));
    s = F::conj(s);
    T* o = Bo + j0 + j + (int64_t)m * N;
    auto put = [&](int slot, E v) {  // slot 0: V2, 1 (or 0): X
      if constexpr (P == 1) {
        o[slot * pl] = v;
      } else {
        o[slot * pl] = v.r;
        o[(kPl + slot) * pl] = v.i;
        o[(2 * kPl + slot) * pl] = -v.i;
        o[(3 * kPl + slot) * pl] = v.r;
      }
    };
    if constexpr (kHess) put(0, Vl[j * kLd + m]);
    put(kPl - 1, s);
  }
}

template <typename T, class F>
__global__ void identity_kernel(int n, T* Z) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * n) return;
  const int i = (int)(idx % n), j = (int)(idx / n);
  F::store(Z + i + (int64_t)j * F::P * n, n, F::real(i == j ? T(1) : T(0)));
}

// C (M x N, ld ldc, imaginary plane `im` rows below) -= A B^T over K columns,
// the planes of C as two batch entries that share A.
template <typename T, class F>
void rank_update(hipStream_t st, int M, int N, int K, const T* A, int64_t lda, const T* B, T* C, int64_t ldc,
                 int64_t im) {
  if (M <= 0 || N <= 0) return;
  const int64_t sB = (int64_t)N * K;
  if constexpr (sizeof(T) == 4)
    gemm_store_f32(st, false, true, M, N, K, A, lda, 0, B, N, sB, C, ldc, im, -1.f, 1.f, F::P, false);
  else
    gemm_store_f64(st, false, true, M, N, K, A, lda, 0, B, N, sB, C, ldc, im, -1.0, 1.0, F::P, false);
}

template <typename T, class F>
void reduce(hipStream_t st, int n, T* H, T* Z, GehrdWork& w) {
  using E = typename F::E;
  constexpr int P = F::P;
  constexpr int KREG = 128 / (int)sizeof(E);
  const int64_t ld = (int64_t)P * n;
  w.nbar = 0;
  hipLaunchKernelGGL((identity_kernel<T, F>), dim3((unsigned)ceil_div((int64_t)n * n, 256)), dim3(256), 0, st, n, Z);
  MSQRT_LAUNCH_CHECK();
  const int nref = n - 2;  // reflectors for columns 0 .. n-3
  if (nref <= 0) return;
  // one workgroup per CU at full LDS
  int ncu = 0, dev = 0;
  MSQRT_HIP(hipGetDevice(&dev));
  MSQRT_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
  // Rows per workgroup: 16 (a quarter of a wave per row sum) until the grid
  // would exceed the co-resident workgroups; small matrices in one workgroup.
  const int gmax = std::min(std::max(1, ncu), kMaxG);
  int rbp = 16;
  while (rbp < kSolo && rbp < n) rbp *= 2;
  if (n > rbp || panel_lds<F>(rbp, n, true) > kLdsMax) {
    rbp = 16;
    while (rbp < kThreads / 2 && ceil_div(n, rbp) > gmax) rbp *= 2;
  }
  // Panels of kNb columns unless the rows per workgroup leave LDS too little
  // room for them (complex double from n = 8193 on, float from 65537 on).
  int nbw = kNb;
  while (nbw > 2 && panel_lds<F>(rbp, n, false, nbw) > kLdsMax) nbw -= 2;
  const int G = (int)ceil_div(n, rbp);
  if (G > gmax || panel_lds<F>(rbp, n, false, nbw) > kLdsMax)
    throw Error{MSQRT_ERR_UNSUPPORTED, "Hessenberg reduction: matrix too large"};
  const bool wf_lds = panel_lds<F>(rbp, n, true, nbw) <= kLdsMax;
  const size_t lds = panel_lds<F>(rbp, n, wf_lds, nbw);
  auto kern = nbw == kNb ? hess_panel_kernel<T, F, KREG, kNb> : hess_panel_kernel<T, F, KREG, 0>;
  MSQRT_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));

  const int npan = (int)ceil_div(nref, nbw);
  const int64_t pl = (int64_t)n * kNb;  // one plane of a panel
  T* Vall = w.V.ensure<T>((int64_t)npan * P * pl);
  T* Tall = w.Tall.ensure<T>((int64_t)npan * P * kNb * kNb);
  T* YV = w.Y.ensure<T>(2 * P * pl);
  T* Bo = w.W.ensure<T>((P == 2 ? 8 : 2) * pl);
  E* ex = w.part.ensure<E>(n + 2 * kMaxG * kNb);
  unsigned* bar = w.bar.ensure<unsigned>(kBarWords);
  if (G > 1) {
    MSQRT_HIP(hipMemsetAsync(bar, 0, sizeof(unsigned) * kBarWords, st));
    w.nbar = 1;
  }
  BarrierBase base{};

  // K-chunks of the V^* products: about four waves per CU, at least one group
  // of k per wave
  auto vta = [&](int K, int N, int N2, const T* V, const T* B, int64_t ldb, int64_t bim, const T* B2,
                 int64_t b2im) {
    constexpr int KG = kWave / Mfma<T>::TM * 4;
    const int tiles = (int)ceil_div(N + N2, 32);
    int by = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(kMaxBy, ceil_div(256, tiles)), ceil_div(K, 4 * KG)));
    const int chunk = (int)ceil_div(ceil_div(K, 4 * by), KG) * KG;
    by = (int)ceil_div(K, 4 * chunk);
    T* Wp = w.W2.ensure<T>((int64_t)by * 4 * P * (N + N2) * kNb);
    hipLaunchKernelGGL((vta_kernel<T, F>), dim3(tiles, by), dim3(256), 0, st, K, chunk, N, N2, V, (int64_t)n, pl,
                       B, ldb, bim, B2, (int64_t)n, b2im, Wp);
    MSQRT_LAUNCH_CHECK();
    return 4 * by;
  };
  // the largest split product first, so the buffer is allocated once
  w.W2.ensure<T>((int64_t)(256 + ceil_div(n + kNb, 32)) * 4 * P * 32 * kNb);

  for (int pi = 0; pi < npan; ++pi) {
    const int p = pi * nbw, nbp = std::min(nbw, nref - p);
    T* V = Vall + (int64_t)pi * P * pl;
    T* Tp = Tall + (int64_t)pi * P * kNb * kNb;
    PanelArgs<T, F> pa{n, p, nbp, rbp, G, nbw, wf_lds ? 1 : 0, H, V, YV, Tp, ex, ex + n, ex + n + kMaxG * kNb, bar, base};
    if (G > 1) {
      void* args[] = {&pa};
      MSQRT_HIP(hipLaunchCooperativeKernel((const void*)kern, dim3(G), dim3(kThreads), args, lds, st));
      const unsigned nb = 2u * (unsigned)nbp - 1u;  // barriers of the launch
      base.gen += nb;
      base.top += (unsigned)std::min(G, 8) * nb;
      for (int g = 0; g < 8 && G > 8; ++g) base.sub[g] += (unsigned)(G / 8 + (g < G % 8 ? 1 : 0)) * nb;
    } else {
      hipLaunchKernelGGL(kern, dim3(1), dim3(kThreads), lds, st, pa);
      MSQRT_LAUNCH_CHECK();
    }
    const int q = p + nbp;
    const int N = n - q, K = n - p - 1;
    const int splits = vta(K, N, kNb, V + p + 1, H + p + 1 + (int64_t)q * ld, ld, n, YV + p + 1, 2 * pl);
    hipLaunchKernelGGL((w2_kernel<T, F, true>), dim3((unsigned)ceil_div(N, 32)), dim3(256), 0, st, splits, N,
                       (const T*)w.W2.as<T>(), (const T*)Tp, (const T*)(V + q), (int64_t)n, pl, Bo);
    MSQRT_LAUNCH_CHECK();
    rank_update<T, F>(st, n, N, 2 * P * kNb, YV, n, Bo, H + (int64_t)q * ld, ld, n);
  }
  // Z(p+1:, p+1:) -= V (T (V^* Z(p+1:, p+1:)))
  for (int pi = npan - 1; pi >= 0; --pi) {
    const int p = pi * nbw, m = n - p - 1;
    const T* V = Vall + (int64_t)pi * P * pl;
    T* Zs = Z + p + 1 + (int64_t)(p + 1) * ld;
    const int splits = vta(m, m, 0, V + p + 1, Zs, ld, n, Zs, n);
    hipLaunchKernelGGL((w2_kernel<T, F, false>), dim3((unsigned)ceil_div(m, 32)), dim3(256), 0, st, splits, m,
                       (const T*)w.W2.as<T>(), (const T*)(Tall + (int64_t)pi * P * kNb * kNb), (const T*)nullptr,
                       (int64_t)0, (int64_t)0, Bo);
    MSQRT_LAUNCH_CHECK();
    rank_update<T, F>(st, m, m, P * kNb, V + p + 1, n, Bo, Zs, ld, n);
  }
}

}  // namespace

template <typename T>
void gehrd(hipStream_t st, int n, T* H, T* Z, GehrdWork& w) {
  reduce<T, HCplx<T>>(st, n, H, Z, w);
}
template <typename T>
void gehrd_real(hipStream_t st, int n, T* H, T* Z, GehrdWork& w) {
  reduce<T, HReal<T>>(st, n, H, Z, w);
}

void gehrd_check(hipStream_t st, GehrdWork& w) {
  if (w.nbar == 0) return;
  unsigned fail = 0;
  MSQRT_HIP(hipMemcpyAsync(&fail, w.bar.as<unsigned>() + kBarFail, sizeof(unsigned), hipMemcpyDeviceToHost, st));
  MSQRT_HIP(hipStreamSynchronize(st));
  if (fail) throw Error{MSQRT_ERR_DEVICE, "Hessenberg reduction: grid barrier timed out"};
}

template void gehrd_real<float>(hipStream_t, int, float*, float*, GehrdWork&);
template void gehrd_real<double>(hipStream_t, int, double*, double*, GehrdWork&);
template void gehrd<float>(hipStream_t, int, float*, float*, GehrdWork&);
template void gehrd<double>(hipStream_t, int, double*, double*, GehrdWork&);

}  // namespace msqrt
