// Device parts of the persistent kernels (persist.hip, adjoint_persist.hip):
// words that are their own flags, bounded waits, and sums in the order of the
// per-iteration launches.
#pragma once

#include "device_math.h"
#include "persist.h"
#include "sweep_common.h"

namespace pncg {

namespace {

typedef unsigned long long u64;
// a NaN that no arithmetic of the kernel produces; a value with these bits
// is published with its last bit flipped
constexpr u64 kEmpty = 0xfff8dead5eef0001ull;

__device__ __forceinline__ u64 ld_agent(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 full(u64 v) { return v == kEmpty ? v ^ 1 : v; }
__device__ __forceinline__ u64 word(double a) { return (u64)__double_as_longlong(a); }
__device__ __forceinline__ double as_double(u64 w) { return __longlong_as_double((long long)w); }
__device__ __forceinline__ float lo_float(u64 w) { return __int_as_float((int)(unsigned)w); }
__device__ __forceinline__ float hi_float(u64 w) { return __int_as_float((int)(unsigned)(w >> 32)); }

// Watches the clock in a polling loop.  A negative limit: the first look that
// finds a word missing is the last.
struct Wait {
  long long t0, limit;
  int n;
  __device__ __forceinline__ Wait(long long l) : t0(0), limit(l), n(0) {}
  // true when the wait has run out
  __device__ __forceinline__ bool over() {
    if ((++n & 63) != 0) return limit < 0;
    const long long t = wall_clock64();
    if (t0 == 0) t0 = t;
    return t - t0 > limit;
  }
};

// The kernel's argument (one struct), to be read from the kernel argument
// segment where it is needed: kept in registers across a whole iteration it
// would spill.  The empty asm statement hides from the compiler that the
// segment is the same each time.
template <typename K>
using ArgPtr = const __attribute__((address_space(4))) K*;
template <typename K>
__device__ __forceinline__ ArgPtr<K> kernel_args() {
  unsigned long long p = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return (ArgPtr<K>)p;
}

// The value again, behind an empty asm statement: what a phase derives from it
// is derived again in the next iteration instead of being kept in registers.
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int fresh_s(int x) {
  x = __builtin_amdgcn_readfirstlane(x);
  asm volatile("" : "+s"(x));
  return x;
}

template <typename T>
__device__ __forceinline__ V3<T> at3(const T* a, int l) { return mk3(a[3 * l], a[3 * l + 1], a[3 * l + 2]); }

// Sum of the values res[N lane] over the lanes [hi - len, hi], all in one row
// of 16, as seg_sum adds them: a balanced tree counted from the last lane.  16
// lanes are read (the words before the first lane of the chunk are other
// arrays of the block's LDS) and those before the run count as zero, so the
// loads have constant offsets and none waits for another.
template <int N, typename R>
__device__ __forceinline__ R row_run_sum(const R* res, int hi, int len) {
  const R* p = res + N * hi;
  R u[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) u[t] = p[-N * t];
#pragma unroll
  for (int t = 1; t < 16; ++t) u[t] = t <= len ? u[t] : R(0);
#pragma unroll
  for (int d = 1; d < 16; d *= 2) {
#pragma unroll
    for (int t = 0; t < 16; t += 2 * d) u[t] += u[t + d];
  }
  return u[0];
}

// The value of the lane whose number differs in bit 0, 1, 2 or 3.
template <int BIT>
__device__ __forceinline__ int lane_xor(int v) {
  if constexpr (BIT == 0) return __builtin_amdgcn_update_dpp(0, v, 0xb1, 0xf, 0xf, false);   // quad_perm [1, 0, 3, 2]
  if constexpr (BIT == 1) return __builtin_amdgcn_update_dpp(0, v, 0x4e, 0xf, 0xf, false);   // quad_perm [2, 3, 0, 1]
  if constexpr (BIT == 2) {
    // shifts by 4 within the row: left into the lower of each two quads, right into the upper
    const int lo = __builtin_amdgcn_update_dpp(0, v, 0x104, 0xf, 0x5, false);
    return __builtin_amdgcn_update_dpp(lo, v, 0x114, 0xf, 0xa, false);
  }
  return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false);                          // row rotated by 8
}
template <int BIT>
__device__ __forceinline__ double lane_xor(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = lane_xor<BIT>((int)b), hi = lane_xor<BIT>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// a summed over lane pairs (BIT) into the lanes with the bit clear, b into the others
template <int BIT>
__device__ __forceinline__ double pair_sums(double a, double b) {
  const bool up = (threadIdx.x >> BIT) & 1;
  return (up ? b : a) + lane_xor<BIT>(up ? a : b);
}
// Sums of six quantities over each row of 16 lanes, in the balanced order of
// wave_sum (neighbouring lanes first).  Halving the number of quantities per
// lane at each step instead of reducing each alone takes 43 instructions
// against 72.  Lane l of a row's first eight (and of the second) receives
// quantity l, for l < 6.
__device__ __forceinline__ double row_sums6(const double (&q)[6]) {
  const double ab = pair_sums<0>(q[0], q[1]), cd = pair_sums<0>(q[2], q[3]), ef = pair_sums<0>(q[4], q[5]);
  const double abcd = pair_sums<1>(ab, cd), ef2 = ef + lane_xor<1>(ef);
  const double all = pair_sums<2>(abcd, ef2);
  return all + lane_xor<3>(all);
}

// Publish quantity q of a logical block: sh holds the wave results [wave][N]
// of its nw waves, added (or compared) in wave order as block_reduce does.
template <int N>
__device__ __forceinline__ void publish(const double* sh, int q, int nw, bool mx, u64* slot) {
  double r = sh[q];
  for (int j = 1; j < nw; ++j) r = mx ? fmax(r, sh[j * N + q]) : r + sh[j * N + q];
  st_agent(slot, full(word(r)));
}

// Wait for the n partials of N quantities (slot [q][n]) and leave the wave
// sums [q][4] in sh: wave w of the four takes partials 64 w + lane and
// 256 + 64 w + lane, the order of reduce_partials.  The loads of a try, and
// those of other() (more words to wait for; true when they have arrived), are
// all in flight together.
template <int N, typename Other>
__device__ __forceinline__ void gather(const u64* slot, int n, unsigned maxmask, double* sh, int nwaves, long long limit,
                                       int* bad, Other&& other) {
  constexpr int T = (N * 4 + 6) / 7;   // tasks of a wave: at least seven waves share N * 4
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
  const int nw = min(4, (n + kWave - 1) / kWave), tasks = N * nw;
  u64 a[T], b[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int t = wave + i * nwaves, j = (t % nw) * kWave + lane;
    a[i] = t < tasks && j < n ? kEmpty : 0;
    b[i] = t < tasks && j + kSBlock < n ? kEmpty : 0;
  }
  Wait w(limit);
  bool odone = false;
  for (;;) {
    // (only the words that have not arrived: polling all of them again would
    // keep the memory busy with 10 MB per try)
    bool ok = true;
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const int t = wave + i * nwaves, q = t / nw, j = (t - q * nw) * kWave + lane;
      if (a[i] == kEmpty) a[i] = ld_agent(slot + q * n + j);
      if (b[i] == kEmpty) b[i] = ld_agent(slot + q * n + j + kSBlock);
    }
    if (!odone) odone = other();
#pragma unroll
    for (int i = 0; i < T; ++i) ok = ok && a[i] != kEmpty && b[i] != kEmpty;
    if (ok && odone) break;
    if (w.over()) {
      *bad = 1;
      break;
    }
  }
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int t = wave + i * nwaves;
    if (t >= tasks) continue;   // uniform over the wave
    const int q = t / nw, j = (t - q * nw) * kWave + lane;
    const bool mx = (maxmask >> q) & 1u;
    double v = 0.0;
    if (j < n) v = mx ? fmax(v, as_double(a[i])) : v + as_double(a[i]);
    if (j + kSBlock < n) v = mx ? fmax(v, as_double(b[i])) : v + as_double(b[i]);
    v = mx ? wave_max(v) : wave_sum(v);
    if (lane == 0) sh[q * 4 + (t - q * nw)] = v;
  }
}
// Totals of N quantities from the wave sums gather() left, by the first wave:
// lane q adds up quantity q, then every lane receives all.
template <int N>
__device__ __forceinline__ void totals(const double* sh, int n, unsigned maxmask, double (&r)[N]) {
  const int nw = min(4, (n + kWave - 1) / kWave), lane = threadIdx.x & (kWave - 1);
  double v = 0.0;
  if (lane < N) {
    const bool mx = (maxmask >> lane) & 1u;
    v = sh[lane * 4];
    for (int w = 1; w < nw; ++w) v = mx ? fmax(v, sh[lane * 4 + w]) : v + sh[lane * 4 + w];
  }
  const long long b = __double_as_longlong(v);
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const int lo = __builtin_amdgcn_readlane((int)b, q), hi = __builtin_amdgcn_readlane((int)(b >> 32), q);
    r[q] = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  }
}

}  // namespace

}  // namespace pncg
