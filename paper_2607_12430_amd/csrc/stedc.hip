// Divide-and-conquer eigensolver for a symmetric tridiagonal matrix
// (Cuppen's tearing, deflation, secular equation, Gu-Eisenstat eigenvectors).
//
// All scalar work (eigenvalues, secular roots, deflation) is float64 on the
// device; the eigenvector matrices and the merge products use the factor
// precision T on MFMA products, the blocks of up to 32 rows in float64.  Every merge of a level is processed by the
// same five launches: one workgroup per merge for the deflation scan, one wave
// per secular root (and per 64 rows for the deflation rotations), per
// recomputed z and per eigenvector, and the products of all merges.  The
// recursion halves every block, so a kernel finds its block from a position
// or a block number alone, and nothing crosses to or from the host between
// levels.  (Block tables copied to the device and the rotation counts read
// back at every level cost more host time than the small levels ran.)
//
// Merge of two solved halves (T1' = Q1 D1 Q1^T, T2' = Q2 D2 Q2^T) coupled by
// beta:  T = diag(Q1, Q2) (D + rho z z^T) diag(Q1, Q2)^T with
// z = [last row of Q1, sign(beta) first row of Q2] / sqrt(2), rho = 2|beta|.
// The merged eigenvectors are diag(Q1, Q2) (after the deflation rotations)
// times M, where M holds the normalised vectors z_i / (d_i - lambda_j) of the
// non-deflated secular problem and unit columns for deflated entries, both
// placed in ascending order of the merged eigenvalues.
#include <algorithm>
#include <climits>
#include <cmath>
#include <vector>

#include "gemm.hpp"
#include "gridsync.hpp"
#include "kernels.hpp"
#include "tridiag.hpp"

namespace msqrt {

namespace {

// Largest leaf.  A leaf's chain of rotations grows with its square (198 us at
// 32), a level of merges costs about 40 us: order 64 takes 0.13 ms with leaves
// of 16, 0.24 with 32; order 1000 0.56 and 0.76.
// A float solve works on blocks of up to 2 kLeaf rows in float64: with the
// merges to 32 rows in float, Z^T Z - I was 10 to 28% larger than with leaves
// of 32.
constexpr int kLeaf = 16;

// A block of the recursion: rows s .. s + m of the concatenated index space;
// a merge (m > kLeaf) has halves of m / 2 and m - m / 2.
struct Block {
  int s, m, id;  // id: entry * 2^depth + path, -1 for no block
  __host__ __device__ int n1() const { return m / 2; }
  __host__ __device__ bool merge() const { return id >= 0 && m > kLeaf; }
};

// Block number id of `depth`.  A leaf met above that depth keeps its place
// with the remaining path bits zero; other paths below it hold nothing.
__host__ __device__ inline Block block_at(int n, int depth, int id) {
  const int e = id >> depth, path = id & ((1 << depth) - 1);
  Block b{e * n, n, id};
  for (int i = depth - 1; i >= 0; --i) {
    if (b.m <= kLeaf) {
      if (path & ((2 << i) - 1)) b.id = -1;
      return b;
    }
    const int h = b.m / 2;
    if (path >> i & 1) {
      b.s += h;
      b.m -= h;
    } else {
      b.m = h;
    }
  }
  return b;
}

// Block of `depth` that holds position p.
__device__ inline Block block_of(int n, int depth, int p) {
  const int e = p / n;
  Block b{e * n, n, e};
  for (int i = 0; i < depth; ++i) {
    b.id <<= 1;
    if (b.m <= kLeaf) continue;
    const int h = b.m / 2;
    if (p >= b.s + h) {
      b.s += h;
      b.m -= h;
      b.id |= 1;
    } else {
      b.m = h;
    }
  }
  return b;
}

// A batch of tridiagonal matrices of order n is solved as one matrix of
// order batch * n whose off-diagonal vanishes at the entry boundaries: every
// position s of the concatenated index space belongs to entry s / n, and no
// leaf or merge straddles two entries.  The eigenvector matrices stay n x n
// per entry (stride n * n); this is the offset of the diagonal block that
// starts at position s.  The float64 blocks of a float solve are kept in a
// band of kBand rows instead (column c of the concatenated space at c * kBand;
// blocks of at most kBand rows do not overlap).
constexpr int kBand = 2 * kLeaf;
template <bool kB>
__device__ inline int64_t blk_off(int s, int n) {
  if (kB) return (int64_t)s * (kBand + 1);
  const int e = s / n, sl = s - e * n;
  return (int64_t)e * n * n + sl + (int64_t)sl * n;
}

// Exponent of an entry whose tridiagonal matrix has an Inf or NaN: its blocks are
// solved as zero matrices, because the merges place columns by comparisons, and
// its eigenvalues are NaN.
constexpr int kNonFinite = INT_MIN;
__device__ inline double scaled_eig(double l, int ex) { return ex == kNonFinite ? NAN : ldexp(l, ex); }

// Per-position metadata arrays (all length n, indexed by s + local index).
struct Meta {
  double* dl;      // non-deflated poles, ascending
  double* zl;      // their z components
  int* cl;         // their original local column
  double* defd;    // deflated eigenvalues, ascending
  int* defc;       // their original local column
  int* rota;       // rotation list: columns a, b
  int* rotb;
  double* rotc;
  double* rots;
  int* kcnt;       // per merge: k, number of deflated, number of rotations
  double* rho;     // per merge
  int* org;        // per root: origin pole index
  double* tau;     // per root: lambda - d_org
  double* lamr;    // per root: lambda
  double* zhat;    // per non-deflated index: recomputed z
  double* tmpd;    // scratch (sorted d), length n
  double* tmpz;    // scratch (sorted z)
  int* tmpc;       // scratch (sorted columns)
};

// ---------------------------------------------------------------------------
// Leaf eigensolver: implicit symmetric QR with Wilkinson shifts on a leaf of
// size L <= kLeaf.  One wave per leaf; every lane runs the scalar recurrence
// redundantly (identical values) and lane r applies the rotations to row r of
// the eigenvector block.  Bound by the dependent chain of one rotation after
// the other, so the chain is kept short: 1/r from the reciprocal square root
// estimate and one cubic Newton step (2^-66 before rounding; the leaf is
// scaled by a power of two so that r^2 cannot overflow, and r^2 close to
// underflow takes hypot), the rotated entries carried in registers, the next
// ones read a step ahead: 150 ns per rotation, 310 with hypot, two divisions
// and LDS reads in the chain.

template <typename T, bool kB>
__global__ __launch_bounds__(64) void leaf_kernel(int depth, const double* dg, const double* eg,
                                                  const int* exs, double* lam, T* Z, int n) {
  __shared__ double d[kLeaf + 2], e[kLeaf + 2], Zl[kLeaf][kLeaf + 3];
  const int lane = threadIdx.x;
  const Block bl = block_at(n, depth, blockIdx.x);
  if (bl.id < 0) return;
  const int s = bl.s, L = bl.m;
  const double d0 = lane < L ? dg[s + lane] : 0.0, e0 = lane + 1 < L ? eg[s + lane] : 0.0;
  const double amax = wave_max(fmax(fabs(d0), fabs(e0)));
  const int ex = amax > 0.0 && amax < INFINITY ? ilogb(amax) : 0;
  if (lane < kLeaf + 2) {
    d[lane] = ldexp(d0, -ex);
    e[lane] = ldexp(e0, -ex);
  }
  if (lane < L)
    for (int c = 0; c < L; ++c) Zl[lane][c] = (c == lane) ? 1.0 : 0.0;
  __syncthreads();
  const double eps = 1.1102230246251565e-16;
  static_assert(kLeaf + 2 <= kWave, "one lane per entry of a leaf");
  const int row = min(lane, kLeaf - 1);
  int hi = L - 1, iters = 0;
  while (hi > 0 && iters < 60 * kLeaf) {
    // lo = 1 + the last negligible e[l] below hi (0 if none): every lane
    // tests its own entry and a ballot finds the last one.  (The entries of
    // the leaf are at most 2; without the absolute term a graded leaf with a
    // zero diagonal never deflates, its shifts underflow.)
    const bool small = lane < hi && fabs(e[lane]) <= eps * (fabs(d[lane]) + fabs(d[lane + 1])) + 1e-140;
    const unsigned long long sm = __ballot(small);
    const int lo = sm ? 64 - __clzll(sm) : 0;
    if (lo == hi) { --hi; continue; }
    ++iters;
    const double dd = (d[hi - 1] - d[hi]) * 0.5;
    const double b2 = e[hi - 1] * e[hi - 1];
    const double den = dd + copysign(sqrt(dd * dd + b2), dd);
    const double mu = (den == 0.0) ? d[hi] : d[hi] - b2 / den;
    double x = d[lo] - mu, z = e[lo];
    double cd = d[lo], ce = z, dk1 = d[lo + 1], ek1 = e[lo + 1];
    double qa = Zl[row][lo], qb = Zl[row][lo + 1];
    for (int k = lo; k < hi; ++k) {
      const double dk2 = d[k + 2], ek2 = e[k + 2], qn = Zl[row][k + 2];
      const double g = fma(x, x, z * z);
      double r, c, sn;
      if (g > 1e-290) {
        const double y0 = __builtin_amdgcn_rsq(g);
        const double er = fma(-g * y0, y0, 1.0);
        const double y = fma(y0 * er, fma(0.375, er, 0.5), y0);
        r = g * y;
        c = x * y;
        sn = z * y;
      } else {
        r = hypot(x, z);
        c = (r == 0.0) ? 1.0 : x / r;
        sn = (r == 0.0) ? 0.0 : z / r;
      }
      // [c s; -s c] [cd ce; ce dk1] [c -s; s c]
      const double p = fma(sn, dk1 - cd, 2.0 * c * ce);
      const double ne = fma(c, p, -ce);
      // Every lane computed the same scalars and writes them itself, so each
      // lane's later reads depend only on its own writes (no barrier).
      if (k > lo) e[k - 1] = r;
      d[k] = fma(sn, p, cd);
      cd = fma(-sn, p, dk1);
      Zl[row][k] = c * qa + sn * qb;
      qa = c * qb - sn * qa;
      const bool more = k + 1 < hi;
      x = ne;
      z = more ? sn * ek1 : 0.0;
      ce = more ? c * ek1 : ne;
      dk1 = dk2;
      ek1 = ek2;
      qb = qn;
    }
    d[hi] = cd;
    e[hi - 1] = ce;
    Zl[row][hi] = qa;
  }
  __syncthreads();
  // Ascending order: rank of eigenvalue c (ties by index).
  __shared__ int rank[kLeaf];
  if (lane < L) {
    int r = 0;
    for (int i = 0; i < L; ++i) r += (d[i] < d[lane]) || (d[i] == d[lane] && i < lane);
    rank[lane] = r;
  }
  __syncthreads();
  if (lane < L) {
    const double l = ldexp(d[lane], ex);
    lam[s + rank[lane]] = depth == 0 ? scaled_eig(l, exs[blockIdx.x]) : l;
    T* Zb = Z + blk_off<kB>(s, n);
    for (int c = 0; c < L; ++c) Zb[lane + (int64_t)rank[c] * (kB ? kBand : n)] = (T)Zl[lane][c];
  }
}

// ---------------------------------------------------------------------------
// Merge preparation: z vector, merge of the two sorted halves, deflation scan.
// One workgroup per merge.

template <typename T, bool kB>
__global__ __launch_bounds__(256) void merge_prep_kernel(int depth, const double* eg, const double* lam,
                                                         const T* Z, int n, Meta mt) {
  const Block g = block_at(n, depth, blockIdx.x);
  if (!g.merge()) return;
  const int s = g.s, n1 = g.n1(), m = g.m, n2 = m - n1;
  const double beta = eg[s + n1 - 1];
  const double sgn = beta >= 0.0 ? 1.0 : -1.0;
  const double rho = 2.0 * fabs(beta);
  const double r2 = 0.7071067811865476;
  const T* Zg = Z + blk_off<kB>(s, n);
  const int ldz = kB ? kBand : n;
  __shared__ double red[4];
  // every position names a column whatever the values are
  for (int i = threadIdx.x; i < m; i += blockDim.x) mt.tmpc[s + i] = i;
  __syncthreads();
  // merge-path placement of the two ascending halves
  double dmax = 0.0, zmax = 0.0;
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    double di, zi;
    int pos;
    if (i < n1) {
      di = lam[s + i];
      zi = r2 * (double)Zg[(n1 - 1) + (int64_t)i * ldz];
      int lo = 0, hi = n2;  // count right values < di
      while (lo < hi) { const int mid = (lo + hi) / 2; if (lam[s + n1 + mid] < di) lo = mid + 1; else hi = mid; }
      pos = i + lo;
    } else {
      const int jr = i - n1;
      di = lam[s + i];
      zi = sgn * r2 * (double)Zg[n1 + (int64_t)i * ldz];
      int lo = 0, hi = n1;  // count left values <= di
      while (lo < hi) { const int mid = (lo + hi) / 2; if (lam[s + mid] <= di) lo = mid + 1; else hi = mid; }
      pos = jr + lo;
    }
    mt.tmpd[s + pos] = di;
    mt.tmpz[s + pos] = zi;
    mt.tmpc[s + pos] = i;
    dmax = fmax(dmax, fabs(di));
    zmax = fmax(zmax, fabs(zi));
  }
  dmax = block_max(dmax, red);
  zmax = block_max(zmax, red);
  __syncthreads();
  // Stage the sorted (d, z, column) triples in LDS for the sequential scan;
  // outputs go straight to global memory (stores only).
  extern __shared__ unsigned char lds_raw[];
  double* d = reinterpret_cast<double*>(lds_raw);
  double* z = d + m;
  int* c = reinterpret_cast<int*>(z + m);
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    d[i] = mt.tmpd[s + i];
    z[i] = mt.tmpz[s + i];
    c[i] = mt.tmpc[s + i];
  }
  __syncthreads();
  __shared__ int counts[3];
  const double eps = 1.1102230246251565e-16;
  const double tol = 8.0 * eps * fmax(dmax, zmax);
  // Rotation test of the scan below for a pair of consecutive survivors
  // (identical arithmetic, so the flags agree with it).
  auto rot_test = [&](double dp, double zp, double dj, double zj) {
    double sn = zp, cs = zj;
    const double tau = hypot(cs, sn);
    const double t = dj - dp;
    cs /= tau;
    sn = -sn / tau;
    return fabs(t * cs * sn) <= tol;
  };
  // Parallel pass: each thread takes a contiguous chunk, survivors of the
  // z-test and deflated entries are placed by block prefix sums, and every
  // pair of consecutive survivors is tested with its original values.  When
  // no pair calls for a rotation this is exactly the scan's result (kept
  // values in order, deflated values ascending); otherwise the sequential
  // scan below redoes the merge.
  __shared__ int scan_k[256], scan_d[256], scan_last[256];
  __shared__ int any_rot;
  const int nt = blockDim.x, tid = threadIdx.x;  // nt <= 256
  const int chunk = (m + nt - 1) / nt, c0 = min(m, tid * chunk), c1 = min(m, c0 + chunk);
  int nk = 0, ndf = 0, last = -1;
  for (int j = c0; j < c1; ++j) {
    if (rho * fabs(z[j]) <= tol) ++ndf;
    else { ++nk; last = j; }
  }
  scan_k[tid] = nk;
  scan_d[tid] = ndf;
  scan_last[tid] = last;
  if (tid == 0) any_rot = 0;
  __syncthreads();
  for (int off = 1; off < nt; off <<= 1) {  // inclusive scans (sum, max)
    const int a = tid >= off ? scan_k[tid - off] : 0, b = tid >= off ? scan_d[tid - off] : 0;
    const int l = tid >= off ? scan_last[tid - off] : -1;
    __syncthreads();
    scan_k[tid] += a;
    scan_d[tid] += b;
    scan_last[tid] = max(scan_last[tid], l);
    __syncthreads();
  }
  {
    int kpos = scan_k[tid] - nk, dpos = scan_d[tid] - ndf;
    int prev = tid > 0 ? scan_last[tid - 1] : -1;
    bool rot = false;
    for (int j = c0; j < c1; ++j) {
      if (rho * fabs(z[j]) <= tol) {
        mt.defd[s + dpos] = d[j];
        mt.defc[s + dpos] = c[j];
        ++dpos;
      } else {
        if (prev >= 0) rot = rot || rot_test(d[prev], z[prev], d[j], z[j]);
        mt.dl[s + kpos] = d[j];
        mt.zl[s + kpos] = z[j];
        mt.cl[s + kpos] = c[j];
        ++kpos;
        prev = j;
      }
    }
    if (rot) any_rot = 1;
  }
  __syncthreads();
  const bool need_scan = any_rot != 0;
  if (!need_scan && tid == 0) {
    counts[0] = scan_k[nt - 1]; counts[1] = scan_d[nt - 1]; counts[2] = 0;
    mt.kcnt[3 * blockIdx.x + 0] = scan_k[nt - 1];
    mt.kcnt[3 * blockIdx.x + 1] = scan_d[nt - 1];
    mt.kcnt[3 * blockIdx.x + 2] = 0;
    mt.rho[blockIdx.x] = rho;
  }
  if (need_scan && tid == 0) {
    int k = 0, nd = 0, nr = 0, pj = -1;
    double dp = 0.0, zp = 0.0;
    int cp = 0;
    for (int j = 0; j < m; ++j) {
      const double dj = d[j], zj = z[j];
      const int cj = c[j];
      if (rho * fabs(zj) <= tol) {
        mt.defd[s + nd] = dj;
        mt.defc[s + nd] = cj;
        ++nd;
        continue;
      }
      if (pj < 0) { pj = j; dp = dj; zp = zj; cp = cj; continue; }
      double sn = zp, cs = zj;
      const double tau = hypot(cs, sn);
      const double t = dj - dp;
      cs /= tau;
      sn = -sn / tau;
      if (fabs(t * cs * sn) <= tol) {
        // Rotate columns pj, j so that z[pj] vanishes; pj deflates.
        mt.rota[s + nr] = cp;
        mt.rotb[s + nr] = cj;
        mt.rotc[s + nr] = cs;
        mt.rots[s + nr] = sn;
        ++nr;
        const double tt = dp * cs * cs + dj * sn * sn;
        const double dnew = dp * sn * sn + dj * cs * cs;
        mt.defd[s + nd] = tt;
        mt.defc[s + nd] = cp;
        ++nd;
        pj = j; dp = dnew; zp = tau; cp = cj;
      } else {
        mt.dl[s + k] = dp;
        mt.zl[s + k] = zp;
        mt.cl[s + k] = cp;
        ++k;
        pj = j; dp = dj; zp = zj; cp = cj;
      }
    }
    if (pj >= 0) {
      mt.dl[s + k] = dp;
      mt.zl[s + k] = zp;
      mt.cl[s + k] = cp;
      ++k;
    }
    counts[0] = k; counts[1] = nd; counts[2] = nr;
    mt.kcnt[3 * blockIdx.x + 0] = k;
    mt.kcnt[3 * blockIdx.x + 1] = nd;
    mt.kcnt[3 * blockIdx.x + 2] = nr;
    mt.rho[blockIdx.x] = rho;
  }
  __syncthreads();
  // Deflated values in ascending order: rank sort in LDS (ties by index).
  // Without rotations they are already in order (d ascending).
  const int nd = counts[1];
  if (need_scan && nd > 1) {
    for (int i = threadIdx.x; i < nd; i += blockDim.x) {
      d[i] = mt.defd[s + i];
      c[i] = mt.defc[s + i];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nd; i += blockDim.x) {
      const double v = d[i];
      int r = 0;
      for (int q = 0; q < nd; ++q) r += (d[q] < v) || (d[q] == v && q < i);
      mt.defd[s + r] = v;
      mt.defc[s + r] = c[i];
    }
  }
}

// Deflation rotations on row p of its merge block.
template <typename T, bool kB>
__device__ inline void merge_rot(const Block& g, int p, const Meta& mt, T* Z, int n) {
  const int nr = mt.kcnt[3 * g.id + 2];
  T* Zr = Z + blk_off<kB>(g.s, n) + (p - g.s);
  const int ldz = kB ? kBand : n;
  for (int q = 0; q < nr; ++q) {
    const int64_t ca = (int64_t)mt.rota[g.s + q] * ldz, cb = (int64_t)mt.rotb[g.s + q] * ldz;
    const double c = mt.rotc[g.s + q], sn = mt.rots[g.s + q];
    const double x = (double)Zr[ca], y = (double)Zr[cb];
    Zr[ca] = (T)(c * x + sn * y);
    Zr[cb] = (T)(c * y - sn * x);
  }
}

// ---------------------------------------------------------------------------
// Secular equation 1/rho + sum_i z_i^2 / (d_i - lambda) = 0, one wave per
// root j (root j lies in (d_j, d_{j+1}), the last one in (d_k, d_k + rho)).
// The root is represented as lambda = d_org + tau with org the nearer pole so
// that d_i - lambda = (d_i - d_org) - tau is computed to high relative
// accuracy.  Iteration: a two-pole rational model fitted to the value and the
// derivatives of the left and right partial sums (Gragg's scheme), solved as
// a quadratic, safeguarded by a bracket that is bisected whenever the model
// step leaves it.

__device__ inline void secular_eval(const double* dl, const double* zl, int k, int org, int j,
                                    double tau, int lane, double& psi, double& phi, double& dpsi,
                                    double& dphi) {
  psi = phi = dpsi = dphi = 0.0;
  const double dorg = dl[org];
  for (int i = lane; i < k; i += kWave) {
    const double del = (dl[i] - dorg) - tau;
    const double w = zl[i] / del;
    if (i <= j) { psi += zl[i] * w; dpsi += w * w; }
    else { phi += zl[i] * w; dphi += w * w; }
  }
  psi = wsum(psi);
  phi = wsum(phi);
  dpsi = wsum(dpsi);
  dphi = wsum(dphi);
}

// Workgroups from N on apply the deflation rotations, 64 rows each.
template <typename T, bool kB>
__global__ __launch_bounds__(64) void secular_kernel(int depth, Meta mt, int n, int N, T* Z) {
  const int w = blockIdx.x;
  const int lane = threadIdx.x;
  if (w >= N) {
    const int p = (w - N) * 64 + lane;
    if (p >= N) return;
    const Block g = block_of(n, depth, p);
    if (g.merge()) merge_rot<T, kB>(g, p, mt, Z, n);
    return;
  }
  const Block g = block_of(n, depth, w);
  if (!g.merge()) return;
  const int b = g.id;
  const int j = w - g.s;
  const int k = mt.kcnt[3 * b];
  if (j >= k) return;
  const double* dl = mt.dl + g.s;
  const double* zl = mt.zl + g.s;
  const double rho = mt.rho[b];
  const double eps = 1.1102230246251565e-16;
  int org;
  double lo, hi, tau;
  if (k == 1) {
    if (lane == 0) {
      mt.org[g.s + j] = 0;
      mt.tau[g.s + j] = rho * zl[0] * zl[0];
      mt.lamr[g.s + j] = dl[0] + rho * zl[0] * zl[0];
    }
    return;
  }
  if (j < k - 1) {
    const double gap = dl[j + 1] - dl[j];
    // f at the midpoint decides the nearer pole
    double psi, phi, dpsi, dphi;
    secular_eval(dl, zl, k, j, j, 0.5 * gap, lane, psi, phi, dpsi, dphi);
    const double fmid = 1.0 / rho + psi + phi;
    if (fmid >= 0.0) { org = j; lo = 0.0; hi = 0.5 * gap; }
    else { org = j + 1; lo = -0.5 * gap; hi = 0.0; }
  } else {
    org = k - 1;
    double zz = 0.0;
    for (int i = lane; i < k; i += kWave) zz += zl[i] * zl[i];
    zz = wsum(zz);
    lo = 0.0;
    hi = rho * zz * (1.0 + 4.0 * eps) + 1e-300;
  }
  tau = 0.5 * (lo + hi);
  for (int it = 0; it < 200; ++it) {
    double psi, phi, dpsi, dphi;
    secular_eval(dl, zl, k, org, j, tau, lane, psi, phi, dpsi, dphi);
    const double f = 1.0 / rho + psi + phi;
    if (f == 0.0) break;
    if (f < 0.0) lo = tau; else hi = tau;
    // convergence: |f| below the rounding level of its terms, or bracket tight
    const double erret = 8.0 * (phi - psi) + 2.0 / rho + fabs(tau) * (dpsi + dphi);
    if (fabs(f) <= eps * erret * 4.0) break;
    if (hi - lo <= 4.0 * eps * fmax(fabs(lo), fabs(hi))) break;
    // model poles relative to the current point
    const double dorg = dl[org];
    const double a0 = (dl[j] - dorg) - tau;  // < 0
    double step_tau;
    bool ok = false;
    if (j < k - 1) {
      const double b0 = (dl[j + 1] - dorg) - tau;  // > 0
      const double s1 = a0 * a0 * dpsi, s2 = b0 * b0 * dphi;
      const double c0 = f - a0 * dpsi - b0 * dphi;
      // c0 eta^2 - B eta + C = 0, eta in (a0, b0)
      const double B = c0 * (a0 + b0) + s1 + s2;
      const double C = c0 * a0 * b0 + s1 * b0 + s2 * a0;
      double eta = 0.0;
      if (c0 == 0.0) {
        if (B != 0.0) { eta = C / B; ok = true; }
      } else {
        const double disc = B * B - 4.0 * c0 * C;
        if (disc >= 0.0) {
          const double q = 0.5 * (B + copysign(sqrt(disc), B));
          const double e1 = q / c0, e2 = (q != 0.0) ? C / q : e1;
          if (e1 > a0 && e1 < b0) { eta = e1; ok = true; }
          else if (e2 > a0 && e2 < b0) { eta = e2; ok = true; }
        }
      }
      step_tau = tau + eta;
    } else {
      const double s1 = a0 * a0 * dpsi;
      const double c0 = f - a0 * dpsi;
      double eta = 0.0;
      if (c0 > 0.0) { eta = a0 + s1 / c0; ok = true; }
      step_tau = tau + eta;
    }
    if (!ok || !(step_tau > lo && step_tau < hi)) {
      // bisection (geometric when the bracket excludes zero)
      if (lo > 0.0 && hi > 0.0 && hi > 4.0 * lo) step_tau = sqrt(lo * hi);
      else if (lo < 0.0 && hi < 0.0 && lo < 4.0 * hi) step_tau = -sqrt(lo * hi);
      else step_tau = 0.5 * (lo + hi);
    }
    if (step_tau == tau) break;
    tau = step_tau;
  }
  if (lane == 0) {
    mt.org[g.s + j] = org;
    mt.tau[g.s + j] = tau;
    mt.lamr[g.s + j] = dl[org] + tau;
  }
}

// Gu-Eisenstat: z_i recomputed from the computed roots so that the computed
// eigenvectors are numerically orthogonal:
//   zhat_i^2 = (lambda_i - d_i)/rho * prod_{j != i} (lambda_j - d_i)/(d_j - d_i).
__global__ __launch_bounds__(64) void lowner_kernel(int depth, Meta mt, int n) {
  const int p = blockIdx.x, lane = threadIdx.x;
  const Block g = block_of(n, depth, p);
  if (!g.merge()) return;
  const int b = g.id;
  const int i = p - g.s;
  const int k = mt.kcnt[3 * b];
  if (i >= k) return;
  const double* dl = mt.dl + g.s;
  const double di = dl[i];
  double prod = 1.0;
  for (int j = lane; j < k; j += kWave) {
    const double lj_di = (dl[mt.org[g.s + j]] - di) + mt.tau[g.s + j];
    prod *= (j == i) ? lj_di / mt.rho[b] : lj_di / (dl[j] - di);
  }
  // product over the wave
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) prod *= __shfl_xor(prod, off, kWave);
  if (lane == 0) {
    const double zh = sqrt(fmax(prod, 0.0));
    mt.zhat[g.s + i] = mt.zl[g.s + i] >= 0.0 ? zh : -zh;
  }
}

// Columns of M: secular eigenvectors (normalised) and unit vectors for the
// deflated entries, at the rank of their eigenvalue; new eigenvalue array.
template <typename T, bool kB>
__global__ __launch_bounds__(64) void vectors_kernel(int depth, Meta mt, const int* exs, T* M, double* lam_new,
                                                     int n) {
  const int w = blockIdx.x, lane = threadIdx.x;
  const Block g = block_of(n, depth, w);
  if (!g.merge()) return;
  const int b = g.id;
  const int q = w - g.s;
  const int k = mt.kcnt[3 * b], nd = mt.kcnt[3 * b + 1];
  T* Mb = M + (int64_t)g.s * (kB ? kBand : n);  // m x m, ld m
  const int m = g.m, ex = depth == 0 ? exs[b] : 0;
  if (q < k) {
    const int j = q;
    const double* dl = mt.dl + g.s;
    const double dorg = dl[mt.org[g.s + j]], tau = mt.tau[g.s + j];
    const double lj = mt.lamr[g.s + j];
    double nrm = 0.0;
    for (int i = lane; i < k; i += kWave) {
      const double v = mt.zhat[g.s + i] / ((dl[i] - dorg) - tau);
      nrm += v * v;
    }
    nrm = sqrt(wsum(nrm));
    // rank among deflated values (strictly smaller)
    int lo = 0, hi = nd;
    while (lo < hi) { const int mid = (lo + hi) / 2; if (mt.defd[g.s + mid] < lj) lo = mid + 1; else hi = mid; }
    T* col = Mb + (int64_t)(j + lo) * m;
    for (int i = lane; i < k; i += kWave) {
      const double v = mt.zhat[g.s + i] / ((dl[i] - dorg) - tau) / nrm;
      col[mt.cl[g.s + i]] = (T)v;
    }
    for (int i = lane; i < nd; i += kWave) col[mt.defc[g.s + i]] = T(0);
    if (lane == 0) lam_new[g.s + j + lo] = scaled_eig(lj, ex);
  } else if (q < k + nd) {
    const int t = q - k;
    const double v = mt.defd[g.s + t];
    int lo = 0, hi = k;  // roots <= v
    while (lo < hi) { const int mid = (lo + hi) / 2; if (mt.lamr[g.s + mid] <= v) lo = mid + 1; else hi = mid; }
    T* col = Mb + (int64_t)(t + lo) * m;
    const int one = mt.defc[g.s + t];
    for (int i = lane; i < m; i += kWave) col[i] = T(i == one ? 1 : 0);
    if (lane == 0) lam_new[g.s + t + lo] = scaled_eig(v, ex);
  }
}

// The products C = A M of a level, A a merge's m x m block of eigenvectors:
// 64 x 64 tiles of every merge in one launch (max_tiles^2 workgroups for
// each block of the level).
// Before the deflation rotations A = diag(Z1, Z2), and a merge that rotated
// no columns keeps that form: tiles within one half then sum over that half
// alone.  A leaf met at this level is copied.  One product launch per merge
// (up to 48 of 10 us at order 1531, full length for batches) was bound by
// launches and by the chain of one 128-tile.
template <typename T, typename TO, bool kB>
__global__ __launch_bounds__(GTHREADS, 2) void merge_gemm_kernel(int depth, int max_tiles, Meta mt, int n,
                                                                 const T* __restrict__ Za, const T* __restrict__ Mm,
                                                                 TO* __restrict__ Zb, const double* lamA,
                                                                 double* lamB) {
  using N = Narrow<T>;
  using M = Mfma<T>;
  extern __shared__ __attribute__((aligned(16))) unsigned char merge_lds[];
  const unsigned per = (unsigned)(max_tiles * max_tiles);
  const int tile = blockIdx.x % per;
  const Block g = block_at(n, depth, blockIdx.x / per);
  if (g.id < 0) return;
  const int m = g.m, t = threadIdx.x;
  const T* A = Za + blk_off<kB>(g.s, n);
  const int ldz = kB ? kBand : n;
  TO* C = Zb + blk_off<false>(g.s, n);
  if (!g.merge()) {
    if (tile > 0) return;
    for (int x = t; x < m * m; x += GTHREADS) C[x % m + (int64_t)(x / m) * n] = (TO)A[x % m + (int64_t)(x / m) * ldz];
    if (t < m) lamB[g.s + t] = lamA[g.s + t];
    return;
  }
  const int tiles = (m + N::NT - 1) / N::NT;
  if (tile >= tiles * tiles) return;
  const int mo = tile % tiles * N::NT, no = tile / tiles * N::NT;
  int k0 = 0, k1 = m;
  if (mt.kcnt[3 * g.id + 2] == 0) {
    if (min(mo + N::NT, m) <= g.n1()) k1 = g.n1();
    else if (mo >= g.n1()) k0 = g.n1();
  }
  constexpr int NBLK = N::NBLK;
  typename M::acc_t acc[NBLK][NBLK];
  const int m0 = max(0, min(mo, m - N::NT)), n0 = max(0, min(no, m - N::NT));
  narrow_product<T, false, false>(A + (int64_t)k0 * ldz, ldz, Mm + (int64_t)g.s * (kB ? kBand : n) + k0, m, m, m, k1 - k0, m0, n0,
                                  reinterpret_cast<T*>(merge_lds), acc);
  const int lane = t % kWave, wave = t / kWave;
#pragma unroll
  for (int i = 0; i < NBLK; ++i)
#pragma unroll
    for (int j = 0; j < NBLK; ++j)
#pragma unroll
      for (int r = 0; r < M::NACC; ++r) {
        const int gi = m0 + wave % 2 * 32 + i * M::TM + M::c_col(lane, r);
        const int gj = n0 + wave / 2 * 32 + j * M::TN + M::c_row(lane, r);
        if (gi >= mo && gj >= no && gi < m && gj < m) C[gi + (int64_t)gj * n] = (TO)acc[i][j][r];
      }
}

// Concatenated float64 copies of the batch's diagonals, torn at every split of
// the recursion (d[q-1] -= |e[q-1]| and d[q] -= |e[q-1]| at split point q);
// the coupling at the end of every entry is zero.  Every entry is scaled by a
// power of two (2^-ex) to entries below 2: the merges compare the poles with
// z, which has norm 1.  One workgroup per entry.
template <typename T>
__global__ __launch_bounds__(1024) void tear_kernel(int n, int depth, const T* d, const T* e, int64_t sD, double* dd,
                                                    double* ee, int* exs) {
  __shared__ double red[1024 / kWave];
  d += blockIdx.x * sD;
  e += blockIdx.x * sD;
  dd += (int64_t)blockIdx.x * n;
  ee += (int64_t)blockIdx.x * n;
  double mx = 0.0;
  auto take = [&](double v) { mx = v <= mx ? mx : v < INFINITY ? v : INFINITY; };  // NaN counts as Inf
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    take(fabs((double)d[i]));
    if (i + 1 < n) take(fabs((double)e[i]));
  }
  mx = block_max(mx, red);
  const bool finite = mx < INFINITY;
  const int ex = mx > 0.0 && finite ? ilogb(mx) : 0;
  if (threadIdx.x == 0) exs[blockIdx.x] = finite ? ex : kNonFinite;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    if (!finite) {
      dd[i] = ee[i] = 0.0;
      continue;
    }
    double v = ldexp((double)d[i], -ex);
    Block bl{0, n, 0};
    for (int l = 0; l < depth && bl.m > kLeaf; ++l) {
      const int q = bl.s + bl.m / 2;
      if (i == q - 1 || i == q) v -= fabs(ldexp((double)e[q - 1], -ex));
      if (i >= q) bl = {q, bl.m - bl.m / 2, 0};
      else bl.m /= 2;
    }
    dd[i] = v;
    ee[i] = (i + 1 < n) ? ldexp((double)e[i], -ex) : 0.0;
  }
}

}  // namespace

template <typename T>
void stedc_batched(hipStream_t st, int n, int batch, const T* d, const T* e, int64_t sD,
                   double* lam, T* Z, StedcWork& w) {
  if (n <= 0 || batch <= 0) return;
  const int64_t nn = (int64_t)n * n;
  const int64_t N64 = (int64_t)n * batch;
  if (N64 > (int64_t)1 << 30 || nn * batch > ((int64_t)1 << 40))
    throw Error{MSQRT_ERR_UNSUPPORTED, "tridiagonal eigensolver: batch too large"};
  const size_t prep_bytes = 2 * sizeof(double) + sizeof(int);  // LDS per row of a merge
  if (n > kLeaf && n * prep_bytes > 140 * 1024)
    throw Error{MSQRT_ERR_UNSUPPORTED, "tridiagonal eigensolver supports n <= 7000"};
  const int N = (int)N64;
  // Static recursion tree of one entry: halve until the pieces are at most
  // kLeaf.  Every entry has the same tree, shifted by a multiple of n.
  int depth = 0;
  auto largest = [&](int dep) { return (int)ceil_div(n, (int64_t)1 << dep); };
  while (largest(depth) > kLeaf) ++depth;

  double* dd = w.dd.ensure<double>(N);
  double* ee = w.ee.ensure<double>(N);
  int* ib = w.rot.ensure<int>((int64_t)10 * N + 16);
  int* exs = ib + 9 * (int64_t)N;
  hipLaunchKernelGGL(tear_kernel<T>, dim3((unsigned)batch), dim3(1024), 0, st, n, depth, d, e, sD, dd, ee, exs);
  MSQRT_LAUNCH_CHECK();
  // the last level writes Z and lam
  T* Z2 = w.Z2.ensure<T>(nn * batch);
  double* lam2 = w.lam.ensure<double>(N);
  T *Za = depth % 2 ? Z2 : Z, *Zb = depth % 2 ? Z : Z2;
  double *lamA = depth % 2 ? lam2 : lam, *lamB = depth % 2 ? lam : lam2;
  auto leaves = [&](auto* z, auto band) {
    using TZ = std::remove_pointer_t<decltype(z)>;
    hipLaunchKernelGGL((leaf_kernel<TZ, decltype(band)::value>), dim3((unsigned)batch << depth), dim3(64), 0, st,
                       depth, dd, ee, exs, lamA, z, n);
    MSQRT_LAUNCH_CHECK();
  };
  if (depth == 0) {
    leaves(Za, std::false_type());
    return;
  }
  MSQRT_HIP(hipMemsetAsync(Za, 0, sizeof(T) * nn * batch, st));
  MSQRT_HIP(hipMemsetAsync(Zb, 0, sizeof(T) * nn * batch, st));

  // metadata buffers, indexed by concatenated position (per merge: by the
  // block number)
  Meta mt;
  double* fb = w.roots.ensure<double>((int64_t)12 * N + 16);
  mt.dl = fb; mt.zl = fb + N; mt.defd = fb + 2 * N; mt.rotc = fb + 3 * N; mt.rots = fb + 4 * N;
  mt.tau = fb + 5 * N; mt.lamr = fb + 6 * N; mt.zhat = fb + 7 * N; mt.tmpd = fb + 8 * N;
  mt.tmpz = fb + 9 * N; mt.rho = fb + 10 * N;
  mt.cl = ib; mt.defc = ib + N; mt.rota = ib + 2 * N; mt.rotb = ib + 3 * N; mt.org = ib + 4 * N;
  mt.tmpc = ib + 5 * N; mt.kcnt = ib + 6 * N;
  // M: the m x m secular eigenvector block of the merge at position s sits
  // at M + s * n (ld m)
  T* M = w.M.ensure<T>(nn * batch);
  // A level: from eigenvectors za (in a band or not) to zb.
  auto level = [&](int dep, auto* za, auto* mm, auto* zb, auto band) {
    using TZ = std::remove_pointer_t<decltype(za)>;
    using TO = std::remove_pointer_t<decltype(zb)>;
    constexpr bool kB = decltype(band)::value;
    const unsigned nb = (unsigned)batch << dep;
    const int mmax = largest(dep);
    gemm_lds_attr(merge_prep_kernel<TZ, kB>, 140 * 1024);
    hipLaunchKernelGGL((merge_prep_kernel<TZ, kB>), dim3(nb), dim3(256), mmax * prep_bytes, st, dep, ee, lamA,
                       (const TZ*)za, n, mt);
    MSQRT_LAUNCH_CHECK();
    hipLaunchKernelGGL((secular_kernel<TZ, kB>), dim3((unsigned)(N + ceil_div(N, 64))), dim3(64), 0, st, dep, mt, n, N,
                       za);
    MSQRT_LAUNCH_CHECK();
    hipLaunchKernelGGL(lowner_kernel, dim3(N), dim3(64), 0, st, dep, mt, n);
    MSQRT_LAUNCH_CHECK();
    hipLaunchKernelGGL((vectors_kernel<TZ, kB>), dim3(N), dim3(64), 0, st, dep, mt, exs, mm, lamB, n);
    MSQRT_LAUNCH_CHECK();
    const int tiles = (int)ceil_div(mmax, Narrow<TZ>::NT);
    gemm_lds_attr(merge_gemm_kernel<TZ, TO, kB>, Narrow<TZ>::kLds);
    hipLaunchKernelGGL((merge_gemm_kernel<TZ, TO, kB>), dim3(nb * tiles * tiles), dim3(GTHREADS), Narrow<TZ>::kLds, st,
                       dep, tiles, mt, n, (const TZ*)za, (const TZ*)mm, zb, (const double*)lamA, lamB);
    MSQRT_LAUNCH_CHECK();
    std::swap(lamA, lamB);
  };
  int dep = depth - 1;
  if constexpr (sizeof(T) == 4) {
    // the first level in float64, its result rounded to float
    double* zd = w.band.ensure<double>((int64_t)2 * N * (kBand + 1));
    MSQRT_HIP(hipMemsetAsync(zd, 0, sizeof(double) * N * (kBand + 1), st));
    leaves(zd, std::true_type());
    level(dep, zd, zd + (int64_t)N * (kBand + 1), Zb, std::true_type());
    std::swap(Za, Zb);
    --dep;
  } else {
    leaves(Za, std::false_type());
  }
  for (; dep >= 0; --dep) {
    level(dep, Za, M, Zb, std::false_type());
    std::swap(Za, Zb);
  }
}

template <typename T>
void stedc(hipStream_t st, int n, const T* d, const T* e, double* lam, T* Z, StedcWork& w) {
  stedc_batched<T>(st, n, 1, d, e, 0, lam, Z, w);
}

template void stedc<float>(hipStream_t, int, const float*, const float*, double*, float*, StedcWork&);
template void stedc<double>(hipStream_t, int, const double*, const double*, double*, double*, StedcWork&);
template void stedc_batched<float>(hipStream_t, int, int, const float*, const float*, int64_t, double*,
                                   float*, StedcWork&);
template void stedc_batched<double>(hipStream_t, int, int, const double*, const double*, int64_t,
                                    double*, double*, StedcWork&);

}  // namespace msqrt
