// Exclusive prefix sums by one workgroup.  Needs kWave, lane_id() and the
// device built-ins (threadIdx, __shfl_up, __syncthreads) from its includer.
#pragma once

#include <stdint.h>

namespace gmp {

// Exclusive prefix sums of f(0..n-1) by one workgroup of kScanThreads threads,
// out[n] the total: tiles of four items a thread, wavefronts scanned with
// shuffles, the wavefront totals by the first wavefront, a running carry.
// lds holds kScanWords words: one per wavefront (its total, then its offset)
// and one for the tile's total, written while slower wavefronts may still read
// their offsets.  Three barriers a tile: a word is written again only after a
// barrier that follows its last reads.
constexpr int kScanThreads = 1024;
constexpr int kScanWaves = kScanThreads / kWave;
constexpr int kScanWords = kScanWaves + 1;
template <typename F>
__device__ inline void block_scan(F &&f, int64_t *out, int64_t n, int64_t *lds) {
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  int64_t carry = 0;
  for (int64_t base = 0; base < n; base += kScanThreads * 4) {
    int64_t v[4];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = base + (int64_t)t * 4 + k;
      v[k] = i < n ? (int64_t)f(i) : 0;
      s += v[k];
    }
    int64_t incl = s;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int64_t y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) lds[w] = incl;
    __syncthreads();
    if (w == 0) {
      const int64_t x = lane < kScanWaves ? lds[lane] : 0;
      int64_t xi = x;
#pragma unroll
      for (int o = 1; o < kScanWaves; o <<= 1) {
        const int64_t y = __shfl_up(xi, o, kWave);
        if (lane >= o) xi += y;
      }
      if (lane < kScanWaves) lds[lane] = xi - x;  // exclusive wavefront offsets
    }
    __syncthreads();
    int64_t ex = carry + lds[w] + (incl - s);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = base + (int64_t)t * 4 + k;
      if (i < n) out[i] = ex;
      ex += v[k];
    }
    if (t == kScanThreads - 1) lds[kScanWaves] = ex - carry;  // the tile's total: the last thread's end
    __syncthreads();
    carry += lds[kScanWaves];
  }
  if (t == 0) out[n] = carry;
}

}  // namespace gmp
