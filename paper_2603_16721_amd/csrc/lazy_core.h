// Wave-level building blocks of the lazy rounds and of the run's counters:
// reductions, sample lists and gene bitmaps (64 genes per lane).  Device code
// only.
#pragma once
#include "dfs_core.h"
#include "pdfs_dev.h"

namespace pdfs {
namespace {

__device__ __forceinline__ int popc64(uint64_t x) { return __popcll((unsigned long long)x); }

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return uniform(v);
}

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
  return uniform(v);
}

// Sum of v over the lanes below this one.
__device__ __forceinline__ int wave_before(int v, int lane) {
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int x = __shfl_up(incl, o, 64);
    if (lane >= o) incl += x;
  }
  return incl - v;
}

__device__ __forceinline__ uint64_t readlane64(uint64_t x, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l);
  return (uint64_t)hi << 32 | lo;
}

// Samples of y (lane k < w64 holds word k) as ids in smp; returns how many.
__device__ __forceinline__ int list_samples(uint64_t y, uint16_t* smp, int lane) {
  const int c = popc64(y);
  int pos = wave_before(c, lane);
  const int m = uniform(__shfl(pos + c, 63, 64));
  wave_lds_sync();   // earlier reads of the list are done
  while (y) {
    smp[pos++] = (uint16_t)(lane * 64 + __builtin_ctzll(y));
    y &= y - 1;
  }
  wave_lds_sync();
  return m;
}

// Bits of word wd inside [lo, hi).
__device__ __forceinline__ uint64_t range_bits(int wd, int lo, int hi) {
  const int b = wd * 64;
  if (b + 64 <= lo || b >= hi) return 0ull;
  uint64_t m = ~0ull;
  if (lo > b) m &= ~0ull << (lo - b);
  if (hi < b + 64) m &= ~(~0ull << (hi - b));
  return m;
}

// First set bit of bm at or after `from` (below nA), or -1.
__device__ __forceinline__ int next_bit(const uint64_t* bm, int from, int nA, int lane) {
  const int w_hi = (nA + 63) >> 6;
  for (int w0 = from >> 6; w0 < w_hi; w0 += 64) {
    const int wd = w0 + lane;
    const uint64_t x = wd < w_hi ? bm[wd] & range_bits(wd, from, nA) : 0ull;
    const unsigned long long any = __ballot(x != 0);
    if (any) {
      const int l = __builtin_ctzll(any);
      const int c = x ? wd * 64 + __builtin_ctzll(x) : 0;
      return uniform(__shfl(c, l, 64));
    }
  }
  return -1;
}

}  // namespace
}  // namespace pdfs
