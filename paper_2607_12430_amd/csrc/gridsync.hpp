// Exchange between the co-resident workgroups of a cooperative launch: coherent
// loads and stores, fixed-order wavefront sums by DPP, values tagged with the
// step they belong to, and a two-level grid barrier (the panel kernels of the
// tridiagonal and Hessenberg reductions).
#pragma once

#include "common.hpp"

namespace msqrt {

constexpr int kSyncThreads = 1024;  // default workgroup size

// Values exchanged between workgroups inside a launch (partial products and
// sums) are written and read with agent-scope atomic stores and loads, which
// are coherent across the XCDs' L2 caches, so the barrier needs no device-wide
// fence: such a fence writes back and invalidates the whole L2 of every XCD
// on every column, and the tiles cached there would be fetched again.
template <typename T>
__device__ inline void cstore(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline T cload(const T* p) {
  return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wavefront sum by DPP: butterflies inside every row of 16 lanes (two quad
// permutations, the half-row mirror, the row mirror) leave each lane with
// its row's sum; the four row sums are then read with readlane.  Every lane
// gets the total (in a fixed order, so results are reproducible).  All 64
// lanes must be active: every call site is reached by whole wavefronts.
template <int CTRL>
__device__ inline int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ inline float dpp_v(float v) {
  return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ inline double dpp_v(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp_i<CTRL>((int)b), hi = dpp_i<CTRL>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ inline float lane_of(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ inline double lane_of(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sum over each row of 16 lanes, left in every lane of the row.
template <typename V>
__device__ inline V rsum16(V v) {
  v += dpp_v<0xB1>(v);
  v += dpp_v<0x4E>(v);
  v += dpp_v<0x141>(v);
  v += dpp_v<0x140>(v);
  return v;
}
template <typename V>
__device__ inline V wsum(V v) {
  v += dpp_v<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_v<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_v<0x141>(v);  // row_half_mirror
  v += dpp_v<0x140>(v);  // row_mirror
  return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}

// Tagged exchange: a value goes out as 64-bit words of 32 bits of it and a
// 32-bit tag (of the step it belongs to), each written and read whole, so a
// reader that finds the tag has the value: the read is the wait, and no store is
// waited for.  A step's words may be overwritten once every workgroup is known
// to have finished reading them.
// The same memory may hold plain floats or doubles from an earlier launch, and
// any finite bit pattern can be one of those (small step numbers are denormal
// floats, which the tails of a kernel matrix have).  A tag is therefore the
// upper half of a NaN, in float as in double, with the step in the payload: no
// finite value and no NaN that arithmetic produces looks like a written word.
typedef unsigned long long tword;
constexpr unsigned kTagSteps = 1u << 19;  // the quiet bit of a double's NaN stays clear
__host__ __device__ constexpr unsigned step_tag(unsigned step) { return 0xFFF00000u + 1u + step; }
template <typename T>
constexpr int kTagW = (int)sizeof(T) / 4;  // words per value
__device__ inline void tag_store(tword* p, float v, unsigned tag) {
  cstore(p, (tword)tag << 32 | __float_as_uint(v));
}
__device__ inline void tag_store(tword* p, double v, unsigned tag) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  cstore(p, (tword)tag << 32 | (unsigned)b);
  cstore(p + 1, (tword)tag << 32 | (unsigned)(b >> 32));
}
template <typename T>
__device__ inline T tag_value(const tword* w) {
  if constexpr (sizeof(T) == 4) return __uint_as_float((unsigned)w[0]);
  else return __longlong_as_double((long long)((unsigned long long)(unsigned)w[1] << 32 | (unsigned)w[0]));
}
// Word at a workgroup-uniform base plus a byte offset of the thread's own.
__device__ inline tword tag_word(const tword* base, unsigned bytes) {
  return cload(reinterpret_cast<const tword*>(reinterpret_cast<const char*>(base) + bytes));
}
// Reads the words load(0 .. N - 1) until all carry the tag in all lanes (a loop
// that lanes leave one by one doubles its registers).  A spin limit keeps a
// broken launch from hanging: it raises the sticky failure flag.
template <int N, class Load>
__device__ __forceinline__ void tag_load(tword (&w)[N], Load load, unsigned tag, unsigned* fail) {
  unsigned spins = 0;
  while (true) {
    bool miss = false;
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = load(k);
#pragma unroll
    for (int k = 0; k < N; ++k) miss = miss || (unsigned)(w[k] >> 32) != tag;
    if (__ballot(miss) == 0) return;
    if ((++spins & 255u) == 0u) {
      if (__ballot(cload(fail) != 0u) != 0) return;
      if (spins > (1u << 24)) {
        cstore(fail, 1u);
        return;
      }
    }
  }
}

// Grid barrier state of one batch entry (unsigned words): the top counter,
// the sticky failure flag, the release word and 8 group counters, each on a
// 256-byte line of its own.
constexpr int kBarTop = 0, kBarFail = 1, kBarRel = 64, kBarSub = 128, kBarSubStride = 64;
constexpr int kBarWords = kBarSub + 8 * kBarSubStride;  // words of one entry's state

// Counter values at the start of a launch.  All counters only grow within one
// reduction, so a barrier needs no reset: the host adds what every launch
// contributes (nothing to the group counters when G <= 8, see grid_arrive).
struct BarrierBase {
  unsigned gen;     // release word: barriers completed
  unsigned top;     // top counter
  unsigned sub[8];  // group counters
};

// Two-level grid barrier, split into arrival and wait so that a workgroup
// can do work that needs no other workgroup's results while the barrier
// completes.  The G workgroups of a batch entry form 8 groups (workgroup
// index mod 8, which is the XCD a workgroup is dispatched to when the entry
// starts on a multiple of 8); a workgroup adds 1 to its group's counter, the
// group's last arrival (known from the value its add returns) adds 1 to the
// top counter, and the last arrival there writes the barrier's generation
// number to the release word, which the other workgroups poll.  Spreading the
// arrivals over 8 counters halves the cost of a barrier of 253 workgroups
// against one shared counter.  Every thread waits for its own coherent
// stores to complete before the workgroup arrives.  The counters are handled
// by the first lane of the last wave (kBarT), which has no row work in the
// tridiagonal kernel, nor in the Hessenberg one with blocks of less than 512
// rows, so the atomics' round trips hold up no thread that has.  A spin limit keeps a
// broken launch from hanging: it raises the sticky failure flag.
template <int NT>
constexpr int kBarT = NT - kWave;

// Arrival; returns true in thread kBarT if this workgroup released barrier k.
template <int NT = kSyncThreads>
__device__ inline bool grid_arrive(unsigned* bar, const BarrierBase& base, unsigned sub_base, int blk,
                                   int G, int k) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // A launch of one workgroup per batch entry synchronises with itself only:
  // the wait above and the workgroup barrier make its stores visible to its
  // own later loads.
  if (G == 1) return true;
  bool released = false;
  if (threadIdx.x == kBarT<NT>) {
    const unsigned g = (unsigned)blk & 7u;
    const unsigned gsz = (unsigned)G / 8u + (g < ((unsigned)G & 7u) ? 1u : 0u);
    const unsigned ng = G < 8 ? (unsigned)G : 8u;
    // with G <= 8 every group has one member, which is always its group's
    // last arrival: its counter is skipped, here and in the host's bases
    const unsigned old =
        G <= 8 ? sub_base + gsz * (unsigned)k - 1u
               : __hip_atomic_fetch_add(&bar[kBarSub + kBarSubStride * g], 1u, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1u == sub_base + gsz * (unsigned)k) {
      const unsigned o2 = __hip_atomic_fetch_add(&bar[kBarTop], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (o2 + 1u == base.top + ng * (unsigned)k) {
        cstore(&bar[kBarRel], base.gen + (unsigned)k);
        released = true;
      }
    }
  }
  return released;
}

// Wait for barrier k (released: what grid_arrive returned).
template <int NT = kSyncThreads>
__device__ inline void grid_wait(unsigned* bar, const BarrierBase& base, int k, bool released) {
  if (threadIdx.x == kBarT<NT> && !released) {
    const unsigned gen = base.gen + (unsigned)k;
    unsigned spins = 0;
    while (cload(&bar[kBarRel]) < gen) {
      __builtin_amdgcn_s_sleep(1);
      if ((++spins & 255u) == 0u) {
        if (cload(&bar[kBarFail]) != 0u) break;
        if (spins > (1u << 24)) {
          cstore(&bar[kBarFail], 1u);
          break;
        }
      }
    }
  }
  __syncthreads();
}

template <int NT = kSyncThreads>
__device__ inline void grid_barrier(unsigned* bar, const BarrierBase& base, unsigned sub_base, int blk,
                                    int G, int k) {
  grid_wait<NT>(bar, base, k, grid_arrive<NT>(bar, base, sub_base, blk, G, k));
}

}  // namespace msqrt
