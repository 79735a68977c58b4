// Multishift QR on an upper Hessenberg matrix with several bulge chains in
// flight: the Schur decomposition of Alg. 2 (complex single shifts,
// CplxRoute) and the real Schur form of the remark on real input in
// Sec. 2.2.1 (Francis double shifts, RealRoute).  GPU-resident; the host
// reads back the active block once per batch of chains.
//
//  * A batch sends K chains of nb bulges through the active block [lo, hi].
//    Chain c runs two windows behind chain c - 1, so at every step the chains
//    work on disjoint diagonal windows of at most W rows: one workgroup per
//    chain chases its bulges through the window in LDS and accumulates the
//    window's transformation U (qr_chase_kernel), then two launches apply all
//    the U to the rest of H and to Z on the matrix cores (qr_apply_kernel).
//  * The shifts of a batch are the eigenvalues of the trailing 2 x 2 diagonal
//    blocks, read by the kernel that tests for deflation.  (Eigenvalues of
//    the whole trailing block save about a tenth of the bulges, but that QR
//    iteration ran before every batch on one workgroup: 250 launches of 166 us at
//    n = 2048 against none.  It runs, as qr_shift_kernel, before the batches of a
//    block that has all but stopped deflating: see schur_qr.)
//  * Within a chain the bulges sit SPAN rows apart and move in lockstep, one
//    row per round: bulge j applies its reflector at position kbase - SPAN j
//    + r in round r.  The reflectors of a round act on disjoint rows and none
//    changes an entry another one is formed from, so all row operations run
//    together, then all column operations.  A wave owns a bulge; of the columns
//    of U that it changes all but one are in registers from the round before.
//  * Blocks of at most W rows are left until the end and finished side by
//    side, one workgroup each, with the same rounds in LDS (qr_small_kernel).
//
// What bounds it: the instructions of a round (16 waves, four to a SIMD) times
// the rounds of a batch; 16 bulges on 128 rows cost 69 us for 79 rows, eight
// 60 us for 103 (with reflectors of one tau; the second part of tau added about
// 5%), so long chains win although their windows advance less.
#pragma once

#include <algorithm>
#include <vector>

#include "gemm.hpp"
#include "schur.hpp"

namespace msqrt {

namespace qr {

constexpr int kThreads = 1024;
constexpr int kNb = kThreads / kWave;  // bulges per chain, one wave each
// Bulges of a batch: a sixth of the active block (a third with single shifts),
// at most kMaxBatch.  A longer batch fills the pipeline of chains better and
// deflates more per pass; past 192 the eigenvalues of the far 2 x 2 blocks are
// too poor as shifts (QR phase at n = 2048: 83, 70, 57, 57 ms for 64, 96, 192,
// 320; complex n = 1024: 54, 51, 42, 42 ms).
constexpr int kMaxBatch = 192;
constexpr int kMaxChains = 13;  // kMaxBatch over the smallest chain_bulges()
constexpr int kPad = 4;      // elements between the H and the U window in LDS
constexpr int kLag = 2;      // windows between consecutive chains of a batch

template <typename T>
__device__ inline T eps_of();
template <> __device__ inline float eps_of<float>() { return 5.9604645e-08f; }
template <> __device__ inline double eps_of<double>() { return 1.1102230246251565e-16; }
template <typename T>
__device__ inline T tiny_of();
template <> __device__ inline float tiny_of<float>() { return 1.1754944e-38f; }
template <> __device__ inline double tiny_of<double>() { return 2.2250738585072014e-308; }

// sqrt(x), 1/x and 1/sqrt(x) for x of ordinary size.  Float: the hardware estimates
// (1 ulp; the IEEE sequences sat on the serial path of every round) with one
// Newton step, without it (rcp_est) only where a common factor cancels.
__device__ inline double root(double x) { return sqrt(x); }
__device__ inline float root(float x) {
  const float r = __builtin_amdgcn_rsqf(x), s = x * r;
  return fmaf(0.5f * r, fmaf(-s, s, x), s);
}
__device__ inline double rcp_of(double x) { return 1.0 / x; }
__device__ inline float rcp_of(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.f), r);
}
__device__ inline double rsq_of(double x) { return 1.0 / sqrt(x); }
__device__ inline float rsq_of(float x) {
  const float r = __builtin_amdgcn_rsqf(x);
  return fmaf(0.5f * r, fmaf(-x * r, r, 1.f), r);
}
__device__ inline double rcp_est(double x) { return 1.0 / x; }
__device__ inline float rcp_est(float x) { return __builtin_amdgcn_rcpf(x); }
// The power of two at or below x > 0, and its reciprocal (x below the largest one).
__device__ inline float pow2_of(float x, float& rcp) {
  const int e = __float_as_int(x) & 0x7f800000;
  rcp = __int_as_float(0x7f000000 - e);
  return __int_as_float(e);
}
__device__ inline double pow2_of(double x, double& rcp) {
  const long long e = __double_as_longlong(x) & 0x7ff0000000000000LL;
  rcp = __longlong_as_double(0x7fe0000000000000LL - e);
  return __longlong_as_double(e);
}

// hi + lo = 2 / (1 + a^2 + b^2) for |a|, |b| <= 1, a^2 + b^2 <= 1 to rounding.
__device__ inline void two_over_norm2(float a, float b, float& hi, float& lo) {
  const double n = fma((double)b, (double)b, fma((double)a, (double)a, 1.0));
  hi = 2.f * __builtin_amdgcn_rcpf((float)n);
  lo = (float)fma(-(double)hi, n, 2.0) * (0.5f * hi);
}
__device__ inline void two_over_norm2(double a, double b, double& hi, double& lo) {
  const double a2 = a * a, b2 = b * b, ea = fma(a, a, -a2), eb = fma(b, b, -b2);
  const double g = fmax(a2, b2), l = fmin(a2, b2);
  const double q = g + l, eq = l - (q - g);
  const double n = 1.0 + q, en = q - (n - 1.0);
  hi = 2.0 / n;
  lo = fma(-hi, en + eq + (ea + eb), fma(-hi, n, 2.0)) * (0.5 * hi);
}

// (1 - a^2 - b^2 - c^2) / 2 for a sum close to 1.
__device__ inline double half_defect(double a, double b, double c) {
  const double a2 = a * a, b2 = b * b, c2 = c * c;
  const double e = fma(a, a, -a2) + fma(b, b, -b2) + fma(c, c, -c2);
  const double g = fmax(b2, c2), l = fmin(b2, c2), q = g + l, eq = l - (q - g);
  const double h = fmax(a2, q), k = fmin(a2, q), n = h + k, en = k - (n - h);
  return 0.5 * ((1.0 - n) - (en + eq + e));
}

// The first lane's value in every lane (as a scalar operand).
__device__ inline float bcast(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ inline double bcast(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <typename T>
__device__ inline cx<T> bcast(cx<T> x) { return {bcast(x.r), bcast(x.i)}; }

template <typename T>
__device__ inline T abs1(T x) { return fabs(x); }
template <typename T>
__device__ inline T abs1(cx<T> x) { return fabs(x.r) + fabs(x.i); }

// Real matrices n x n, ld n; double shifts; reflectors
// P = I - tau v v^T, v = (1, w1, w2).
template <typename TT>
struct RealRoute {
  using T = TT;
  using E = TT;
  static constexpr bool kComplex = false;
  static constexpr int SPAN = 3;
  static constexpr int W = sizeof(T) == 4 ? 128 : 96;
  static constexpr int kFinal = 2;  // order of the blocks the iteration leaves
  struct Refl { T tau, w1, w2, tl; };  // tau + tl = 2 / v^T v
  // Shift pair: the eigenvalues of [[a, b], [c, d]].  Its sum and product would do,
  // but next to a diagonal that agrees with them to half the digits (a cluster, a
  // defective eigenvalue) the first column below would be their rounding.
  struct Shift { T a, d, bc; };
  __host__ __device__ static int64_t ldim(int n) { return n; }
  __device__ static E load(const T* p, int64_t) { return p[0]; }
  __device__ static void store(T* p, int64_t, E v) { p[0] = v; }
  __device__ static E zero() { return T(0); }
  __device__ static E one() { return T(1); }

  // P x = (beta, 0, 0); x[2] = 0 for a two-element reflector.  x is scaled by a
  // power of two near its largest entry, so neither a subnormal nor a huge bulge
  // over- or underflows; entries below the smallest normal number count as zero.
  // beta replaces a subdiagonal entry once per bulge, so its errors must have
  // mean zero: the hardware's estimates were 0.29 units low on average, which
  // drifts over the bulges that pass (A = 71 I + G, n = 4096, float: backward
  // error 1.26 times that of the fewer bulges before, now 0.70; n = 2048, QR
  // phase: float 59.3 -> 60.7 ms, double, without the division by the largest
  // entry and with one square root, 226 -> 204).
  // tau = 2 / v^T v is formed from the rounded v, so P is orthogonal whatever
  // the error of v, and with its own rounding error tl beside it: an error
  // eps of tau makes P^T P = I + 4 eps v v^T / v^T v, the same for every row
  // and column that P is applied to, which is more than the rounding of
  // the application itself.  Many bulges with the shifts of 2 x 2 blocks are
  // 1.6 times the bulges of single chains with better shifts, and the error
  // had grown with them.  n = 2048, ||Z^T Z - I||_F: float 4.0e-4 without tl,
  // 2.6e-4 with it (3.2e-4 with the fewer bulges), double 1.1e-12, 7.5e-13
  // (9.4e-13); for 8% of the QR phase (float 54.7 -> 59.3 ms).
  __device__ static Refl make(const E (&x)[3], E& beta) {
    T rs;
    const T sc = pow2_of(fmax(fabs(x[0]), fmax(fabs(x[1]), fabs(x[2]))), rs);
    const T a = x[0] * rs, b = x[1] * rs, c = x[2] * rs;
    const T t = b * b + c * c;
    if (!(sc >= tiny_of<T>() * T(4)) || t == T(0)) {
      beta = x[0];
      return {T(0), T(0), T(0), T(0)};
    }
    const T n2 = a * a + t;
    const T nrm = root(n2);
    const T den = a + copysign(nrm, a);
    const T id = rcp_of(den);
    const T w1 = b * id, w2 = c * id;
    beta = -copysign(nrm, a) * sc;
    T tau, tl;
    two_over_norm2(w1, w2, tau, tl);
    return {tau, w1, w2, tl};
  }
  // first column of (H - s1 I)(H - s2 I) at the top row l of the active block
  __device__ static void intro(const E* h, int ldh, int l, Shift sh, E (&x)[3]) {
    const T h00 = h[l + l * ldh], h10 = h[l + 1 + l * ldh], h01 = h[l + (l + 1) * ldh];
    const T h11 = h[l + 1 + (l + 1) * ldh], h21 = h[l + 2 + (l + 1) * ldh];
    const T p = h00 - sh.a, q = h00 - sh.d;
    x[0] = p * q - sh.bc + h01 * h10;
    x[1] = h10 * (p + (h11 - sh.d));
    x[2] = h10 * h21;
  }
  __device__ static void rows(Refl f, E (&y)[3]) {
    const T d = y[0] + f.w1 * y[1] + f.w2 * y[2];
    const T s = fma(f.tau, d, f.tl * d);
    y[0] -= s;
    y[1] -= s * f.w1;
    y[2] -= s * f.w2;
  }
  __device__ static void cols(Refl f, E (&y)[3]) { rows(f, y); }
  // shift pair q from the q-th trailing 2 x 2 block [[a, b], [c, d]]
  __device__ static Shift shift(int, E a, E b, E c, E d) { return {a, d, b * c}; }
  // shift pairs from the quasi-triangular h of order m, the last blocks first; two
  // real eigenvalues make a pair
  __device__ static int eigen_shifts(const E* h, int ldh, int m, Shift* out) {
    int cnt = 0;
    bool single = false;
    T x = T(0);
    for (int k = m - 1; k >= 0;) {
      const T d = h[k + k * ldh];
      if (k > 0 && h[k + (k - 1) * ldh] != T(0)) {
        out[cnt++] = shift(0, h[k - 1 + (k - 1) * ldh], h[k - 1 + k * ldh], h[k + (k - 1) * ldh], d);
        k -= 2;
      } else {
        if (single) out[cnt++] = {x, d, T(0)};
        single = !single;
        x = d;
        k -= 1;
      }
    }
    if (single) out[cnt++] = {x, x, T(0)};
    return cnt;
  }
  __device__ static int shift_block(int q) { return q; }
  __device__ static Shift exceptional(int q, E d, T e) {
    const T re = d + (q % 2 ? -e : e) * T(0.75) * T(1 + q % 3), im = T(0.5) * e;
    return {re, re, -im * im};
  }
  // bulges of an in-LDS sweep / of a batch on an active block of order m
  __host__ __device__ static int small_bulges(int m) { return m / 6 < 1 ? 1 : (m / 6 > kNb ? kNb : m / 6); }
  __host__ __device__ static int batch_bulges(int m) {
    return m / 6 > kMaxBatch ? kMaxBatch : m / 6;
  }
};

// Complex matrices in the stacked layout (ld 2n, imaginary plane n rows
// below); single shifts; rotations G = [c s; -conj(s) c], c real,
// H <- G H G^*, U <- U G^*.
template <typename TT>
struct CplxRoute {
  using T = TT;
  using E = cx<TT>;
  static constexpr bool kComplex = true;
  static constexpr int SPAN = 2;
  static constexpr int W = sizeof(T) == 4 ? 96 : 64;
  static constexpr int kFinal = 1;
  struct Refl { T c; cx<T> s; T h; };  // (1 + h) [c s; -conj(s) c] is unitary
  using Shift = cx<TT>;
  __host__ __device__ static int64_t ldim(int n) { return 2 * (int64_t)n; }
  __device__ static E load(const T* p, int64_t ld) { return {p[0], p[ld / 2]}; }
  __device__ static void store(T* p, int64_t ld, E v) {
    p[0] = v.r;
    p[ld / 2] = v.i;
  }
  __device__ static E zero() { return {T(0), T(0)}; }
  __device__ static E one() { return {T(1), T(0)}; }

  // G [f; g] = [r; 0].  c and s do not change when f and g are scaled
  // together, so both are divided by max(|f|_1, |g|_1) first; with q =
  // |f|^2 (|f|^2 + |g|^2), c = |f|^2 / sqrt(q) and s = f conj(g) / sqrt(q).
  // In double the defect of c^2 + |s|^2 goes along as h, as tl does in the real
  // route (n = 1024, ||Z^* Z - I||_F: 5.0e-13 without, 3.2e-13 with, 3.2e-13
  // before there were several chains); the float rotation is without it well
  // within what it was with hypot (1.7e-4 against 3.2e-3).
  __device__ static Refl make(const E (&x)[2], E& beta) {
    const E f = x[0], g = x[1];
    const T ag = abs1(g), sc = fmax(abs1(f), ag);
    if (!(ag > tiny_of<T>()) || !(sc > tiny_of<T>() * T(4))) {
      beta = f;
      return {T(1), zero(), T(0)};
    }
    const T rs = rcp_est(sc);
    const E fs = cscale(f, rs), gs = cscale(g, rs);
    const T f2 = cabs2(fs), g2 = cabs2(gs);
    Refl o;
    if (f2 < (sizeof(T) == 4 ? T(1e-24) : T(1e-200))) {  // |f| far below u |g|
      const T r = rsq_of(g2);
      o = {T(0), cscale(cconj(gs), r), T(0)};
    } else {
      const T r = rsq_of(f2 * (f2 + g2));
      o = {f2 * r, cscale(cmul(fs, cconj(gs)), r), T(0)};
    }
    if constexpr (sizeof(T) == 8) o.h = half_defect(o.c, o.s.r, o.s.i);
    beta = cadd(cscale(f, o.c), cmul(o.s, g));
    return o;
  }
  __device__ static void intro(const E* h, int ldh, int l, Shift sh, E (&x)[2]) {
    x[0] = csub(h[l + l * ldh], sh);
    x[1] = h[l + 1 + l * ldh];
  }
  __device__ static E unit(Refl f, E a) {
    if constexpr (sizeof(T) == 8) return {fma(f.h, a.r, a.r), fma(f.h, a.i, a.i)};
    else return a;
  }
  __device__ static void rows(Refl f, E (&y)[2]) {
    const E a = cadd(cscale(y[0], f.c), cmul(f.s, y[1]));
    y[1] = unit(f, csub(cscale(y[1], f.c), cmulc(f.s, y[0])));
    y[0] = unit(f, a);
  }
  __device__ static void cols(Refl f, E (&y)[2]) {
    const E a = cadd(cscale(y[0], f.c), cmul(y[1], cconj(f.s)));
    y[1] = unit(f, csub(cscale(y[1], f.c), cmul(y[0], f.s)));
    y[0] = unit(f, a);
  }
  // shift q: an eigenvalue of the (q / 2)-th trailing 2 x 2 block
  // [[a, b], [c, d]], the one closer to d for even q
  __device__ static Shift shift(int q, E a, E b, E c, E d) {
    const E p = cscale(csub(a, d), T(0.5));
    const E disc = csqrt_principal(cadd(cmul(p, p), cmul(b, c)));
    const E mid = cscale(cadd(a, d), T(0.5));
    const E l1 = cadd(mid, disc), l2 = csub(mid, disc);
    const bool first = abs1(csub(l1, d)) <= abs1(csub(l2, d));
    return first == (q % 2 == 0) ? l1 : l2;
  }
  __device__ static int eigen_shifts(const E* h, int ldh, int m, Shift* out) {
    for (int k = 0; k < m; ++k) out[k] = h[m - 1 - k + (m - 1 - k) * ldh];
    return m;
  }
  __device__ static int shift_block(int q) { return q / 2; }
  __device__ static Shift exceptional(int q, E d, T e) {
    return {d.r + (q % 2 ? -e : e) * T(0.75) * T(1 + q % 3), d.i + T(0.5) * e};
  }
  __host__ __device__ static int small_bulges(int m) { return m / 3 < 1 ? 1 : (m / 3 > kNb ? kNb : m / 3); }
  __host__ __device__ static int batch_bulges(int m) {
    return m / 3 > kMaxBatch ? kMaxBatch : m / 3;
  }
};

// Negligible subdiagonal entry: below ulp times the two adjacent diagonal
// entries, or below ulp ||H||_F.  A perturbation of that size is within the
// backward error the factorisation has anyway, and without the norm-wise
// floor subdiagonals next to eigenvalues much smaller than ||H|| can stall
// above the local threshold in float32 (seen with one large outlier
// eigenvalue, e.g. a uniform(0, 1) matrix plus shift).
template <typename E, typename T>
__device__ inline bool negligible(E sub, E d0, E d1, T hnorm) {
  const T a = abs1(sub), ulp = eps_of<T>();
  return a <= ulp * (abs1(d0) + abs1(d1)) || a <= fmax(tiny_of<T>() * T(1e4), ulp * hnorm);
}

// Keeps a loaded value where it was loaded: without a use outside the lane
// predicate the compiler sinks the load into the predicated store and its
// latency adds to the next one's.
__device__ inline void pin(float& x) { asm volatile("" : "+v"(x)); }
__device__ inline void pin(double& x) { asm volatile("" : "+v"(x)); }
template <typename T>
__device__ inline void pin(cx<T>& x) {
  pin(x.r);
  pin(x.i);
}

// One bulge's share of a round, first half: the reflector on rows c0 ..
// c0+NR-1 (c0 = k + 1) from column k, or from the shift when it enters, and
// the row operation on the columns right of k, RI per lane.
template <class A, int NR, int RI>
__device__ __forceinline__ typename A::Refl row_step(typename A::E* h, int wl, int k, int lo,
                                                     const typename A::Shift* sh, int lane) {
  using E = typename A::E;
  constexpr int S = A::SPAN, LD = A::W + 1;
  const int c0 = k + 1;
  E* const row = h + c0;
  E y[RI][S], x[S];
  int off[RI];
#pragma unroll
  for (int e = 0; e < RI; ++e) {
    off[e] = __mul24(min(c0 + lane + kWave * e, A::W - 1), LD);
#pragma unroll
    for (int q = 0; q < S; ++q) y[e][q] = q < NR ? row[off[e] + q] : A::zero();
  }
  if (k < lo) {
    A::intro(h, LD, lo, *sh, x);
  } else {
#pragma unroll
    for (int q = 0; q < S; ++q) x[q] = q < NR ? row[q + k * LD] : A::zero();
  }
#pragma unroll
  for (int e = 0; e < RI; ++e)
#pragma unroll
    for (int q = 0; q < NR; ++q) pin(y[e][q]);
  E beta;
  const typename A::Refl f = A::make(x, beta);
  if (lane == 0 && k >= lo) {
    row[k * LD] = beta;
#pragma unroll
    for (int q = 1; q < NR; ++q) row[q + k * LD] = A::zero();
  }
#pragma unroll
  for (int e = 0; e < RI; ++e) {
    A::rows(f, y[e]);
    if (c0 + lane + kWave * e < wl) {
#pragma unroll
      for (int q = 0; q < NR; ++q) row[off[e] + q] = y[e][q];
    }
  }
  return f;
}

// Second half: the column operation on rows 0 .. r1 of H and on U.  Of the
// columns c0 .. c0+SPAN-1 of U all but the last are in ua from the bulge's
// round before (loaded here if this is its first); the column that the bulge
// leaves is stored (all of them if it is its last).  RI rows per lane; ua is
// rolled on for all of them, so a lane's second row finds zeros there (the
// columns of U are zero in rows that far down) when its turn comes.
template <class A, int NR, int RI>
__device__ __forceinline__ void col_step(typename A::E* h, typename A::E* u, int c0, int r1,
                                         const typename A::Refl f,
                                         typename A::E (&ua)[(A::W + kWave - 1) / kWave][A::SPAN], bool first,
                                         bool last, int wl, int lane) {
  using E = typename A::E;
  constexpr int S = A::SPAN, LD = A::W + 1;
  E* const hc = h + c0 * LD;
  E* const uc = u + c0 * LD;
  E y[RI][S];
  if (first) {
#pragma unroll
    for (int e = 0; e < RI; ++e)
#pragma unroll
      for (int q = 0; q + 1 < S; ++q) ua[e][q] = uc[min(lane + kWave * e, A::W - 1) + q * LD];
  }
#pragma unroll
  for (int e = 0; e < RI; ++e) {
    const int i = min(lane + kWave * e, A::W - 1);
#pragma unroll
    for (int q = 0; q < S; ++q) y[e][q] = q < NR ? hc[i + q * LD] : A::zero();
    ua[e][S - 1] = NR == S ? uc[i + (S - 1) * LD] : A::zero();
  }
#pragma unroll
  for (int e = 0; e < RI; ++e) {
#pragma unroll
    for (int q = 0; q < NR; ++q) pin(y[e][q]);
    if (NR == S) pin(ua[e][S - 1]);
  }
#pragma unroll
  for (int e = 0; e < RI; ++e) {
    const int i = lane + kWave * e;
    A::cols(f, y[e]);
    if (i <= r1) {
#pragma unroll
      for (int q = 0; q < NR; ++q) hc[i + q * LD] = y[e][q];
    }
    A::cols(f, ua[e]);
    if (i < wl) {
      uc[i] = ua[e][0];
      if (last) {
#pragma unroll
        for (int q = 1; q < NR; ++q) uc[i + q * LD] = ua[e][q];
      }
    }
#pragma unroll
    for (int q = 0; q + 1 < S; ++q) ua[e][q] = ua[e][q + 1];
  }
}

// The rounds between a bulge's first and last: the same two halves without
// any test.  A round is bound by instruction issue (one wave64 vector
// instruction per SIMD and 2 ns, four waves to a SIMD), so everything that a
// round could test is arranged to hold:
//  * the row operation starts at column k itself, whose entries the first
//    lane has, so the reflector's vector comes from there;
//  * lanes past the last column work on the padding between h and u;
//  * the column operation runs over all rows: below the bulge H is zero, and
//    so is U (see rounds), and rows past the window are never written back;
//  * RR and RC (column and row items per lane) are fixed per call.
// rowb: byte offset of (k + 1, k + lane); colb: of (lane, k + 1).  (Float,
// window of 128: with the tests a round took 0.61 us for one bulge and 1.08 us
// for 16, here 0.32 and 0.75 us.)
template <class A, int RR, int RC>
__device__ __forceinline__ void steady_rounds(char* hb, char* ub, int& rowb, int& colb, int count,
                                              typename A::E (&ua)[(A::W + kWave - 1) / kWave][A::SPAN],
                                              int lane) {
  using E = typename A::E;
  constexpr int S = A::SPAN, W = A::W, LD = W + 1, B = sizeof(E), kPadB = W * LD * B;
  auto at = [](char* p, int off) -> E& { return *reinterpret_cast<E*>(p + off); };
#pragma clang loop unroll(disable)
  for (; count > 0; --count) {
    E y[RR][S], x[S], z[RC][S];
    int ro[RR];
#pragma unroll
    for (int e = 0; e < RR; ++e) {
      ro[e] = min(rowb + e * kWave * LD * B, kPadB);
#pragma unroll
      for (int q = 0; q < S; ++q) y[e][q] = at(hb, ro[e] + q * B);
    }
#pragma unroll
    for (int q = 0; q < S; ++q) x[q] = bcast(y[0][q]);
    E beta;
    const typename A::Refl f = A::make(x, beta);
#pragma unroll
    for (int e = 0; e < RR; ++e) A::rows(f, y[e]);
    if (lane == 0) {
      y[0][0] = beta;
#pragma unroll
      for (int q = 1; q < S; ++q) y[0][q] = A::zero();
    }
#pragma unroll
    for (int e = 0; e < RR; ++e)
#pragma unroll
      for (int q = 0; q < S; ++q) at(hb, ro[e] + q * B) = y[e][q];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < RC; ++e) {
      if (kWave * (e + 1) > W && lane >= W - kWave * e) break;
#pragma unroll
      for (int q = 0; q < S; ++q) z[e][q] = at(hb, colb + (kWave * e + q * LD) * B);
      ua[e][S - 1] = at(ub, colb + (kWave * e + (S - 1) * LD) * B);
    }
#pragma unroll
    for (int e = 0; e < RC; ++e) {
      if (kWave * (e + 1) > W && lane >= W - kWave * e) break;
      A::cols(f, z[e]);
#pragma unroll
      for (int q = 0; q < S; ++q) at(hb, colb + (kWave * e + q * LD) * B) = z[e][q];
      A::cols(f, ua[e]);
      at(ub, colb + kWave * e * B) = ua[e][0];
#pragma unroll
      for (int q = 0; q + 1 < S; ++q) ua[e][q] = ua[e][q + 1];
    }
    rowb += (LD + 1) * B;
    colb += LD * B;
    __syncthreads();
  }
}

// Rounds 0..R-1 of a chain of nb bulges on the LDS window h (order wl) with
// its transformation u; lo and hi are the ends of the active block in window
// coordinates (either may lie outside).  Wave j has bulge j, which enters at
// k = lo - 1 (its first reflector comes from shift j) and leaves after
// k = hi - 2, where a reflector of the real route has two rows.  kFresh: u
// starts as the identity.  A column of U then reaches S - 1 rows further down
// with every bulge that has passed it, and one row per lane suffices until
// row kWave is reached.  Called by the whole workgroup; ends with a barrier.
template <class A, bool kFresh>
__device__ __forceinline__ void rounds(typename A::E* h, typename A::E* u, int wl, int kbase, int R, int lo,
                                       int hi, int nb, const typename A::Shift* sh) {
  using E = typename A::E;
  constexpr int S = A::SPAN, W = A::W, LD = W + 1, RI = (W + kWave - 1) / kWave, B = sizeof(E);
  const int j = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  // rounds [ra, rb) in which this wave's bulge moves
  const int k0 = kbase - S * j;
  const int ra = min(R, max(0, lo - 1 - k0)), rb = j < nb ? max(ra, min(R, hi - 1 - k0)) : ra;
  E ua[RI][S];
#pragma unroll
  for (int e = 0; e < RI; ++e)
#pragma unroll
    for (int q = 0; q < S; ++q) ua[e][q] = A::zero();
  auto idle = [](int n) {
    for (; n > 0; --n) {
      __syncthreads();
      __syncthreads();
    }
  };
  // the bulge's first and last round in this call
  auto single = [&](int r) {
    const int k = k0 + r;
    const bool full = S == 2 || k < hi - 2;
    const typename A::Refl f = full ? row_step<A, S, RI>(h, wl, k, lo, sh + j, lane)
                                    : row_step<A, 2, RI>(h, wl, k, lo, sh + j, lane);
    __syncthreads();
    const int r1 = min(min(k + S + 1, hi), wl - 1);
    if (full) col_step<A, S, RI>(h, u, k + 1, r1, f, ua, r == ra, r == rb - 1, wl, lane);
    else col_step<A, 2, RI>(h, u, k + 1, r1, f, ua, r == ra, r == rb - 1, wl, lane);
    __syncthreads();
  };
  idle(ra);
  if (rb > ra) single(ra);
  if (rb > ra + 1) {
    int k = k0 + ra + 1;
    const int ke = k0 + rb - 1;
    int rowb = (k + 1 + (k + lane) * LD) * B, colb = (lane + (k + 1) * LD) * B;
    char *hb = reinterpret_cast<char*>(h), *ub = reinterpret_cast<char*>(u);
    if constexpr (RI == 1) {
      steady_rounds<A, 1, 1>(hb, ub, rowb, colb, ke - k, ua, lane);
    } else {
      // the row operation needs a second item per lane before k1, the column
      // operation from k2 on
      const int k1 = min(ke, max(k, wl - kWave)), k2 = min(ke, max(k, kFresh ? kWave - 1 - S - (S - 1) * j : k));
      const int km = min(k1, k2), kx = max(k1, k2);
      steady_rounds<A, 2, 1>(hb, ub, rowb, colb, km - k, ua, lane);
      if (k1 > k2) steady_rounds<A, 2, 2>(hb, ub, rowb, colb, kx - km, ua, lane);
      else steady_rounds<A, 1, 1>(hb, ub, rowb, colb, kx - km, ua, lane);
      steady_rounds<A, 1, 2>(hb, ub, rowb, colb, ke - kx, ua, lane);
    }
    single(rb - 1);
  }
  idle(R - rb);
}

// Window load / store.  Entries below the band-th subdiagonal are zero.
template <class A>
__device__ __forceinline__ void win_load(typename A::E* h, typename A::E* u, const typename A::T* H, int64_t ld,
                                int s, int m, int band) {
  using E = typename A::E;
  constexpr int W = A::W, N = (W * W + kThreads - 1) / kThreads;
  E v[N];
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int x = threadIdx.x + kThreads * e, i = x % W, j = x / W;
    v[e] = (i < m && j < m && i <= j + band) ? A::load(H + (s + i) + (int64_t)(s + j) * ld, ld) : A::zero();
  }
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int x = threadIdx.x + kThreads * e, i = x % W, j = x / W;
    if (i < m && j < m) {
      h[i + j * (W + 1)] = v[e];
      u[i + j * (W + 1)] = i == j ? A::one() : A::zero();
    }
  }
}

// U is written for qr_apply_kernel's registers: its operand fragments one after
// the other (32 columns; block of TM columns; group of KG rows; lane; four
// rows), so that a wave reads each with consecutive 16-byte loads.  Planes
// real, then imaginary; zero outside m x m.
template <class A>
__device__ __forceinline__ void win_store(const typename A::E* h, const typename A::E* u, typename A::T* H,
                                 int64_t ld, int s, int m, int band, typename A::T* U) {
  using M = Mfma<typename A::T>;
  constexpr int W = A::W, TM = M::TM, NB = 32 / TM, KG = kWave / TM * 4, G = W / KG;
  for (int x = threadIdx.x; x < W * W; x += kThreads) {
    const int i = x % W, j = x / W;
    if (i < m && j < m)
      A::store(H + (s + i) + (int64_t)(s + j) * ld, ld, i <= j + band ? h[i + j * (W + 1)] : A::zero());
  }
  for (int x = threadIdx.x; x < W * W; x += kThreads) {
    const int lane = x / 4 % kWave, f = x / (4 * kWave);  // fragment (32-column block, b, g)
    const int i = f % G * KG + lane / TM * 4 + x % 4;
    const int j = f / (G * NB) * 32 + f / G % NB * TM + lane % TM;
    A::store(U + x, 2 * W * W, i < m && j < m ? u[i + j * (W + 1)] : A::zero());
  }
}
template <class A>
constexpr int64_t u_elems() { return (int64_t)A::W * A::W * (A::kComplex ? 2 : 1); }

// Bulges of a chain: at most one per wave, and few enough that a chain gains
// at least half a window per step, so that windows kLag apart do not overlap.
template <class A>
constexpr int chain_bulges() {
  static_assert(kLag == 2, "half a window per step");
  return std::min(kNb, (A::W - 2) / (2 * A::SPAN));
}

// One window of a chain at one step of a batch.
struct ChainWin {
  int s, wl, kbase, R, sh0;  // first row, order, position of bulge 0 in round 0, rounds, first shift
};
template <typename T>
struct ChaseArgs {
  int n, lo, hi, nb;
  T* H;
  T* U;
  const T* shifts;
  ChainWin w[kMaxChains];
};

// One workgroup per chain: load the window, run its rounds, write it back
// with U.
template <class A>
__global__ __launch_bounds__(kThreads) void qr_chase_kernel(ChaseArgs<typename A::T> a) {
  using E = typename A::E;
  constexpr int W = A::W;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  E* h = reinterpret_cast<E*>(smem);
  E* u = h + (W + 1) * W + kPad;
  __shared__ typename A::Shift sh[kNb];
  const ChainWin w = a.w[blockIdx.x];
  const int64_t ld = A::ldim(a.n);
  if (threadIdx.x < a.nb) sh[threadIdx.x] = reinterpret_cast<const typename A::Shift*>(a.shifts)[w.sh0 + threadIdx.x];
  win_load<A>(h, u, a.H, ld, w.s, w.wl, A::SPAN);
  __syncthreads();
  rounds<A, true>(h, u, w.wl, w.kbase - w.s, w.R, a.lo - w.s, a.hi - w.s, a.nb, sh);
  win_store<A>(h, u, a.H, ld, w.s, w.wl, A::SPAN, a.U + blockIdx.x * u_elems<A>());
}

// Rotation G = [[c, -s], [s, c]] that brings the 2x2 block [[a, b], [e, d]]
// one step towards standard form under G^T M G:
//   real eigenvalues (((a - d)/2)^2 + b e >= 0): the first column of G is an
//     eigenvector, so the rotated block is upper triangular;
//   complex pair: 2 theta solves (a - d) cos 2t + (b + e) sin 2t = 0, the
//     difference of the rotated diagonal entries, which then agree.
// Returns 0 when the block already is in standard form, 1 for the real case,
// 2 for the complex case.
template <typename T>
__device__ inline int std_rotation(T a, T b, T e, T d, T& c, T& s) {
  c = T(1);
  s = T(0);
  if (e == T(0)) return 0;
  const T sc = fmax(fmax(fabs(a - d), fabs(b)), fabs(e));
  const T p = T(0.5) * (a - d) / sc;
  const T disc = p * p + (b / sc) * (e / sc);
  if (disc >= T(0)) {
    const T r = sqrt(disc);
    const T lm = p + (p >= T(0) ? r : -r);  // (lambda - d) / sc
    const T es = e / sc;
    const T nrm = sqrt(lm * lm + es * es);
    c = lm / nrm;
    s = es / nrm;
    return 1;
  }
  if (a == d) return 0;  // equal diagonal and b e < 0
  const T u = (a - d) / sc, v = (b + e) / sc;
  const T r = sqrt(u * u + v * v);
  const T c2 = v / r, s2 = -u / r;
  if (c2 >= T(0)) {
    c = sqrt(T(0.5) * (T(1) + c2));
    s = s2 / (T(2) * c);
  } else {
    s = sqrt(T(0.5) * (T(1) - c2));
    if (s2 < T(0)) s = -s;
    c = s2 / (T(2) * s);
  }
  return 2;
}

// Standardises every 2x2 diagonal block of the quasi-triangular LDS matrix h
// (order m) and accumulates the rotations in u.  The blocks' rotations act on
// disjoint index pairs, so all row operations run together, then all column
// operations; three passes at most (the second and third remove rounding).
template <class A>
__device__ __forceinline__ void standardize_all(typename A::E* h, typename A::E* u, int m) {
  using T = typename A::T;
  constexpr int LD = A::W + 1;
  __shared__ T rc[A::W], rs[A::W];
  __shared__ int kind[A::W];
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  for (int pass = 0; pass < 3; ++pass) {
    int kd = 0;
    if (t < A::W) {
      T c = T(1), s = T(0);
      if (t + 1 < m)
        kd = std_rotation(h[t + t * LD], h[t + (t + 1) * LD], h[t + 1 + t * LD], h[t + 1 + (t + 1) * LD], c, s);
      rc[t] = c;
      rs[t] = s;
      kind[t] = kd;
    }
    if (!__syncthreads_or(kd)) return;
    for (int p = wave; p + 1 < m; p += kThreads / kWave) {
      if (kind[p] == 0) continue;
      for (int c = p + lane; c < m; c += kWave) {
        const T x = h[p + c * LD], y = h[p + 1 + c * LD];
        h[p + c * LD] = rc[p] * x + rs[p] * y;
        h[p + 1 + c * LD] = -rs[p] * x + rc[p] * y;
      }
    }
    __syncthreads();
    for (int p = wave; p + 1 < m; p += kThreads / kWave) {
      if (kind[p] == 0) continue;
      for (int x = lane; x < p + 2 + m; x += kWave) {
        T* q = (x < p + 2 ? h + x : u + (x - p - 2)) + p * LD;
        const T y0 = q[0], y1 = q[LD];
        q[0] = rc[p] * y0 + rs[p] * y1;
        q[LD] = -rs[p] * y0 + rc[p] * y1;
      }
    }
    __syncthreads();
    if (kd == 1) {
      h[t + 1 + t * LD] = T(0);
    } else if (kd == 2) {
      const T avg = T(0.5) * (h[t + t * LD] + h[t + 1 + (t + 1) * LD]);
      h[t + t * LD] = avg;
      h[t + 1 + (t + 1) * LD] = avg;
    }
    __syncthreads();
  }
}

// (Quasi-)triangular form of the LDS block h (order m) with u: sweeps of up to
// kNb bulges; a wave finds the split points of the whole block by ballots, so
// every wave knows them without an exchange.  Shifts from several 2 x 2 blocks
// can go round in circles (a block of 3 I + the cyclic permutation of order 600
// did, in double); a block that has not deflated for kPatience sweeps gets the
// one from its last 2 x 2 block.  Returns false when the iteration limit is hit.
constexpr int kPatience = 20;
template <class A>
__device__ __forceinline__ bool lds_schur(typename A::E* h, typename A::E* u, int m, typename A::T hnorm,
                                          typename A::Shift* sh) {
  using T = typename A::T;
  using E = typename A::E;
  constexpr int W = A::W, LD = W + 1;
  static_assert(W <= 2 * kWave, "two ballots cover a block");
  const int lane = threadIdx.x % kWave;
  const bool w0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave) == 0;
  const int itmax = 30 * max(10, m);
  int hi = m - 1, its = 0, total = 0;
  for (;;) {
    // split points: bit k of the mask is set when block boundary k | k-1 is
    // negligible (bit 0 always)
    unsigned long long mask[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int k = lane + kWave * e;
      bool neg = k == 0;
      if (k >= 1 && k <= hi) {
        neg = negligible<E, T>(h[k + (k - 1) * LD], h[k - 1 + (k - 1) * LD], h[k + k * LD], hnorm);
        if (neg && w0) h[k + (k - 1) * LD] = A::zero();
      }
      mask[e] = __ballot(neg);
    }
    int l = 0;
    const int hi0 = hi;
    while (hi >= 0) {
      const unsigned long long up = hi >= kWave ? mask[1] & (~0ull >> (2 * kWave - 1 - hi)) : 0ull;
      const unsigned long long dn = hi >= kWave ? mask[0] : mask[0] & (~0ull >> (kWave - 1 - hi));
      l = up ? 2 * kWave - 1 - __builtin_clzll(up) : kWave - 1 - __builtin_clzll(dn);
      if (hi - l + 1 > A::kFinal) break;
      hi = l - 1;
    }
    hi = __builtin_amdgcn_readfirstlane(hi);
    l = __builtin_amdgcn_readfirstlane(l);
    if (hi < 0) return true;
    its = hi == hi0 ? its + 1 : 1;
    if (++total > itmax) return false;
    const int nb = its > kPatience ? 1 : A::small_bulges(hi - l + 1);
    if ((int)threadIdx.x < nb) {
      const int q = threadIdx.x, p = hi - 2 * A::shift_block(q);
      typename A::Shift v = A::shift(q, h[p - 1 + (p - 1) * LD], h[p - 1 + p * LD], h[p + (p - 1) * LD], h[p + p * LD]);
      if (its % 10 == 0) {
        T e = abs1(h[hi + (hi - 1) * LD]);
        if (hi - 2 >= l) e += abs1(h[hi - 1 + (hi - 2) * LD]);
        v = A::exceptional(2 * q, h[hi + hi * LD], e);
      }
      sh[q] = v;
    }
    __syncthreads();
    rounds<A, false>(h, u, m, l - 1, hi - l + A::SPAN * (nb - 1), l, hi, nb, sh);
  }
}

// Finishes the diagonal blocks list[2 b], list[2 b + 1] = first row, order
// (at most W), b < *cnt: (quasi-)triangular form with U.
template <class A>
__global__ __launch_bounds__(kThreads) void qr_small_kernel(int n, typename A::T* H, const int* list,
                                                            const int* cnt, typename A::T* U,
                                                            int* status, typename A::T hnorm) {
  using E = typename A::E;
  constexpr int W = A::W;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  E* h = reinterpret_cast<E*>(smem);
  E* u = h + (W + 1) * W + kPad;
  __shared__ typename A::Shift sh[kNb];
  const int b = blockIdx.x;
  if (b >= cnt[0]) return;
  const int s = list[2 * b], m = list[2 * b + 1];
  const int64_t ld = A::ldim(n);
  win_load<A>(h, u, H, ld, s, m, 1);
  __syncthreads();
  const bool ok = lds_schur<A>(h, u, m, hnorm, sh);
  __syncthreads();
  if (!ok && threadIdx.x == 0) atomicOr(status, 1);
  if constexpr (!A::kComplex) standardize_all<A>(h, u, m);
  win_store<A>(h, u, H, ld, s, m, A::kFinal - 1, U + b * u_elems<A>());
}

// Shifts of a batch as the eigenvalues of the trailing block of order m (rows
// s ..) of the active block; H is only read.  One workgroup.  The shifts stay as
// they are if that block does not converge.
template <class A>
__global__ __launch_bounds__(kThreads) void qr_shift_kernel(int n, typename A::T* H, int s, int m,
                                                            typename A::T* shifts, typename A::T hnorm) {
  using E = typename A::E;
  constexpr int W = A::W, LD = W + 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  E* h = reinterpret_cast<E*>(smem);
  E* u = h + (W + 1) * W + kPad;
  __shared__ typename A::Shift sh[kNb], list[A::W];
  __shared__ int cnt;
  win_load<A>(h, u, H, A::ldim(n), s, m, 1);
  __syncthreads();
  const bool ok = lds_schur<A>(h, u, m, hnorm, sh);
  __syncthreads();
  if (!ok) return;
  if (threadIdx.x == 0) cnt = A::eigen_shifts(h, LD, m, list);
  __syncthreads();
  typename A::Shift* sp = reinterpret_cast<typename A::Shift*>(shifts);
  for (int q = threadIdx.x; q < kMaxChains * kNb; q += kThreads) sp[q] = list[q % cnt];
}

// Deflation test on rows 0..hi0 of H, one workgroup.  Negligible subdiagonal
// entries are set to zero; trailing blocks of at most W rows leave the active
// matrix and are appended to the list of finished ranges (consecutive blocks
// share a range while it has at most W rows).  out: {hi, lo} of the active
// block that remains (hi = -1: none), out[2] = number of ranges.  Then the
// shifts of the next batch; exceptional ones when `ex` is set and the active
// block is still [lo0, hi0].
template <class A>
__global__ __launch_bounds__(kThreads) void qr_scan_kernel(int n, typename A::T* H, int hi0, int lo0,
                                                           int ex, int* out, int* list,
                                                           typename A::T* shifts, typename A::T hnorm) {
  using T = typename A::T;
  using E = typename A::E;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned* mask = reinterpret_cast<unsigned*>(smem);
  __shared__ int act[2];
  const int64_t ld = A::ldim(n);
  const int nw = hi0 / 32 + 1;
  for (int x = threadIdx.x; x < nw; x += kThreads) mask[x] = x == 0 ? 1u : 0u;
  __syncthreads();
  for (int k = 1 + threadIdx.x; k <= hi0; k += kThreads) {
    T* p = H + k + (int64_t)(k - 1) * ld;
    if (negligible<E, T>(A::load(p, ld), A::load(p - 1, ld), A::load(p + ld, ld), hnorm)) {
      A::store(p, ld, A::zero());
      atomicOr(&mask[k / 32], 1u << (k % 32));
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int hi = hi0, lo = 0, cnt = out[2];
    while (hi >= 0) {
      int w = hi / 32;
      unsigned v = mask[w] & (~0u >> (31 - hi % 32));
      while (v == 0u) v = mask[--w];
      lo = 32 * w + 31 - __builtin_clz(v);
      if (hi - lo + 1 > A::W) break;
      if (cnt > 0 && list[2 * cnt - 2] + list[2 * cnt - 1] - lo <= A::W) {
        list[2 * cnt - 1] += list[2 * cnt - 2] - lo;
        list[2 * cnt - 2] = lo;
      } else {
        list[2 * cnt] = lo;
        list[2 * cnt + 1] = hi - lo + 1;
        ++cnt;
      }
      hi = lo - 1;
    }
    out[0] = hi;
    out[1] = lo;
    out[2] = cnt;
    act[0] = hi;
    act[1] = lo;
  }
  __syncthreads();
  const int hi = act[0], lo = act[1];
  if (hi < 0) return;
  const int nb = A::batch_bulges(hi - lo + 1);
  typename A::Shift* sp = reinterpret_cast<typename A::Shift*>(shifts);
  // the last chain may be partly filled past nb: its shifts repeat
  for (int q0 = threadIdx.x; q0 < kMaxChains * kNb; q0 += kThreads) {
    const int q = q0 % nb, p = hi - 2 * A::shift_block(q);
    const T* d = H + p + (int64_t)p * ld;
    typename A::Shift v = A::shift(q, A::load(d - 1 - ld, ld), A::load(d - 1, ld), A::load(d - ld, ld), A::load(d, ld));
    if (ex && hi == hi0 && lo == lo0) {
      const T* c = H + hi + (int64_t)hi * ld;
      v = A::exceptional(q, A::load(c, ld), abs1(A::load(c - ld, ld)));
    }
    sp[q0] = v;
  }
}

// The windows' transformations applied to the rest of H and to Z, one
// launch per side (blockIdx.y = window, from w[] or from the device list):
//   rows: H(s : s+wl, s+wl : n) <- U^* H(...)      panels of 32 columns
//   cols: H(0 : s, s : s+wl) <- H(...) U, Z(:, s : s+wl) <- Z(...) U
//                                                   panels of 32 rows
// The panel is staged in LDS, k-contiguous; wave v forms 32 of the W
// outputs of every panel line on MFMA, its part of U held in registers.  The
// operand whose index is the contiguous one of the output goes second, so the
// stores are coalesced.  (n = 2048: 25 us per step for one window on the
// vector units with U copied to every workgroup's LDS; 22 us for up to 13
// windows here.)
struct WinRange { int s, wl; };
template <typename T>
struct ApplyArgs {
  int n;
  T* H;
  T* Z;
  const T* U;
  const int* list;
  const int* cnt;
  WinRange w[kMaxChains];
};

template <class A, bool kCols>
__global__ __launch_bounds__(A::W / 32 * kWave) void qr_apply_kernel(ApplyArgs<typename A::T> a) {
  using T = typename A::T;
  using E = typename A::E;
  using M = Mfma<T>;
  constexpr int W = A::W, P = A::kComplex ? 2 : 1, NT = W / 32 * kWave;
  constexpr int LDP = W + 16 / (int)sizeof(T);
  constexpr int TM = M::TM, NB = 32 / TM, KG = kWave / TM * 4, G = W / KG;
  static_assert(W % KG == 0 && W % 32 == 0, "whole groups of k and whole output blocks");
  __shared__ __attribute__((aligned(16))) T pnl[P][32 * LDP];
  const int n = a.n, y = blockIdx.y;
  if (a.list && y >= a.cnt[0]) return;
  const int s = a.list ? a.list[2 * y] : a.w[y].s, wl = a.list ? a.list[2 * y + 1] : a.w[y].wl;
  const int64_t ld = A::ldim(n);
  // panel: element (line c, k) at base + c * lstr + k * kstr
  T* base;
  int nl;
  int64_t lstr, kstr;
  if (!kCols) {
    const int c0 = s + wl + 32 * (int)blockIdx.x;
    nl = min(32, n - c0);
    base = a.H + s + (int64_t)c0 * ld;
    lstr = ld;
    kstr = 1;
  } else {
    const int gZ = (n + 31) / 32;
    const bool z = (int)blockIdx.x < gZ;
    const int r0 = 32 * (z ? (int)blockIdx.x : (int)blockIdx.x - gZ);
    nl = min(32, (z ? n : s) - r0);
    base = (z ? a.Z : a.H) + r0 + (int64_t)s * ld;
    lstr = 1;
    kstr = ld;
  }
  if (nl <= 0) return;
  const int t = threadIdx.x, lane = t % kWave, ib = t / kWave * 32;
  const int mn = lane % TM, kk = lane / TM;
  const T* U = a.U + y * u_elems<A>();
  T uf[P][NB][G][4];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const T* q = U + p * W * W + ((((ib / 32) * NB + b) * G + g) * kWave + lane) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) uf[p][b][g][e] = q[e];
      }
  constexpr int N = (32 * W + NT - 1) / NT;
  static_assert(N * NT == 32 * W, "panel split");
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int x = t + NT * e;
    const int c = kCols ? x % 32 : x / W, k = kCols ? x / 32 : x % W;
    E v = A::zero();
    if (c < nl && k < wl) v = A::load(base + c * lstr + k * kstr, ld);
    if constexpr (A::kComplex) {
      pnl[0][c * LDP + k] = v.r;
      pnl[1][c * LDP + k] = v.i;
    } else {
      pnl[0][c * LDP + k] = v;
    }
  }
  __syncthreads();
  typename M::acc_t acc[P][NB][NB];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int c = 0; c < NB; ++c) acc[p][b][c] = typename M::acc_t{};
  const T sg = kCols ? T(1) : T(-1);  // U or conj(U)
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      T pf[P][4];
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) pf[p][e] = pnl[p][(c * TM + mn) * LDP + g * KG + 4 * kk + e];
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          auto mac = [&](typename M::acc_t& d, T uv, T pv) { d = kCols ? M::mma(uv, pv, d) : M::mma(pv, uv, d); };
          mac(acc[0][b][c], uf[0][b][g][e], pf[0][e]);
          if constexpr (A::kComplex) {
            const T ui = sg * uf[1][b][g][e];
            mac(acc[0][b][c], -ui, pf[1][e]);
            mac(acc[1][b][c], uf[0][b][g][e], pf[1][e]);
            mac(acc[1][b][c], ui, pf[0][e]);
          }
        }
    }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int r = 0; r < M::NACC; ++r) {
        const int i = ib + b * TM + (kCols ? M::c_row(lane, r) : M::c_col(lane, r));
        const int l = c * TM + (kCols ? M::c_col(lane, r) : M::c_row(lane, r));
        if (i < wl && l < nl) {
          T* o = base + l * lstr + i * kstr;
          o[0] = acc[0][b][c][r];
          if constexpr (A::kComplex) o[ld / 2] = acc[1][b][c][r];
        }
      }
}

template <class A>
constexpr size_t win_lds() { return sizeof(typename A::E) * ((size_t)(A::W + 1) * A::W * 2 + kPad); }

template <class A>
void launch_apply(hipStream_t st, const ApplyArgs<typename A::T>& a, int windows) {
  const int g = (int)ceil_div(a.n, 32);
  hipLaunchKernelGGL((qr_apply_kernel<A, false>), dim3(g, windows), dim3(A::W / 32 * kWave), 0, st, a);
  MSQRT_LAUNCH_CHECK();
  hipLaunchKernelGGL((qr_apply_kernel<A, true>), dim3(2 * g, windows), dim3(A::W / 32 * kWave), 0, st, a);
  MSQRT_LAUNCH_CHECK();
}

// (Quasi-)triangular Schur form of the Hessenberg matrix H, Z <- Z U.
template <class A>
bool schur_qr(hipStream_t st, int n, typename A::T* H, typename A::T* Z, HseqrWork& w,
              typename A::T hnorm) {
  using T = typename A::T;
  constexpr int W = A::W;
  if (n <= 0) return true;
  gemm_lds_attr(qr_small_kernel<A>, win_lds<A>());
  gemm_lds_attr(qr_chase_kernel<A>, win_lds<A>());
  gemm_lds_attr(qr_shift_kernel<A>, win_lds<A>());
  // two neighbouring finished ranges together have more than W rows
  const int max_ranges = 2 * n / W + 2;
  T* U = w.U.ensure<T>(std::max(max_ranges, kMaxChains) * u_elems<A>());
  T* shifts = w.shifts.ensure<T>(sizeof(typename A::Shift) / sizeof(T) * kMaxChains * kNb);
  int* flag = w.flag.ensure<int>(8);  // [0] status, [4..6] the scan's result
  int* list = w.scratch.ensure<int>(2 * max_ranges);
  MSQRT_HIP(hipMemsetAsync(flag, 0, sizeof(int) * 8, st));
  ApplyArgs<T> aa{};
  aa.n = n;
  aa.H = H;
  aa.Z = Z;
  aa.U = U;
  int hi = n - 1, lo = 0, batches = 0, stuck = 0;
  std::vector<int> ends;  // hi of every batch
  const int max_batches = 30 * std::max(10, n / 16) + 100;
  for (;;) {
    const bool ex = stuck > 0 && stuck % 6 == 0;  // exceptional shifts if the block stays
    hipLaunchKernelGGL(qr_scan_kernel<A>, dim3(1), dim3(kThreads), sizeof(unsigned) * (hi / 32 + 1), st, n,
                       H, hi, lo, ex ? 1 : 0, flag + 4, list, shifts, hnorm);
    MSQRT_LAUNCH_CHECK();
    int res[2];
    MSQRT_HIP(hipMemcpyAsync(res, flag + 4, sizeof(res), hipMemcpyDeviceToHost, st));
    MSQRT_HIP(hipStreamSynchronize(st));
    if (res[0] < 0) break;
    stuck = (batches > 0 && res[0] == hi && res[1] == lo) ? stuck + 1 : 0;
    hi = res[0];
    lo = res[1];
    if (++batches > max_batches || stuck > 300) return false;  // no progress: give up
    int total = A::batch_bulges(hi - lo + 1);
    // Shifts from separate 2 x 2 blocks are poor when the trailing block is close to
    // a multiple of an orthogonal matrix (3 I + a cyclic permutation): then the
    // eigenvalues of the whole trailing block, which cost as much as a few batches
    // (float 0.3, complex double 0.9 ms), once six batches have deflated less than a
    // sixteenth of the eigenvalues they aimed at.  The permutation of order 256 in
    // double 63 -> 40 ms.  Double factors of random matrices pass through such
    // stretches as well; there the phase moved by -4 to +5% (orders 256 to 2048; with
    // a quarter instead of a sixteenth it was 3% longer at n = 2048, and the
    // permutation of order 1024 took 201 instead of 185 ms).
    ends.push_back(hi);
    constexpr int kLook = 6;  // batches
    const int eigs = total * (A::kComplex ? 1 : 2);
    const bool poor = batches > 10 && 16 * (ends[ends.size() - 1 - kLook] - hi) < eigs;
    if (poor && !ex) {
      const int ms = 3 * kNb;
      static_assert(3 * kNb <= W, "the block fits a window");
      hipLaunchKernelGGL(qr_shift_kernel<A>, dim3(1), dim3(kThreads), win_lds<A>(), st, n, H, hi - ms + 1, ms, shifts,
                         hnorm);
      MSQRT_LAUNCH_CHECK();
      total = std::min(total, A::kComplex ? ms : ms / 2);
    }
    const int K = (int)ceil_div(total, chain_bulges<A>()), nb = (int)ceil_div(total, K);
    // the windows of one chain; bulge j sits at kbase - SPAN j
    std::vector<ChainWin> win;
    int s = lo, kb = lo - 1;
    for (;;) {
      const int e = std::min(s + W - 1, hi);
      const int R = e < hi ? (e - A::SPAN - 1) - kb + 1 : hi - 2 - kb + A::SPAN * (nb - 1) + 1;
      win.push_back({s, e - s + 1, kb, R, 0});
      if (e == hi) break;
      kb += R;
      s = kb - A::SPAN * (nb - 1);
    }
    const int nwin = (int)win.size();
    ChaseArgs<T> ca{};
    ca.n = n;
    ca.lo = lo;
    ca.hi = hi;
    ca.nb = nb;
    ca.H = H;
    ca.U = U;
    ca.shifts = shifts;
    for (int t = 0; t < nwin + kLag * (K - 1); ++t) {
      int act = 0;
      for (int c = 0; c < K; ++c) {
        const int i = t - kLag * c;
        if (i < 0 || i >= nwin) continue;
        ca.w[act] = win[i];
        ca.w[act].sh0 = c * nb;
        aa.w[act] = {win[i].s, win[i].wl};
        ++act;
      }
      hipLaunchKernelGGL(qr_chase_kernel<A>, dim3(act), dim3(kThreads), win_lds<A>(), st, ca);
      MSQRT_LAUNCH_CHECK();
      launch_apply<A>(st, aa, act);
    }
  }
  hipLaunchKernelGGL(qr_small_kernel<A>, dim3(max_ranges), dim3(kThreads), win_lds<A>(), st, n, H,
                     (const int*)list, (const int*)(flag + 6), U, flag, hnorm);
  MSQRT_LAUNCH_CHECK();
  aa.list = list;
  aa.cnt = flag + 6;
  launch_apply<A>(st, aa, max_ranges);
  int hflag = 0;
  MSQRT_HIP(hipMemcpyAsync(&hflag, flag, sizeof(int), hipMemcpyDeviceToHost, st));
  MSQRT_HIP(hipStreamSynchronize(st));
  return hflag == 0;
}

}  // namespace qr

}  // namespace msqrt
