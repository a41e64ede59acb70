// Listing the points in reach of a node tile in LDS, for the Gaussian fits.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mls {

// The input arrays are global memory.  Said explicitly, their loads are
// global loads also where the compiler cannot see it (parameters read from
// memory in the served batches) instead of flat loads, which also wait on
// the LDS counter.
template <typename V>
__device__ __forceinline__ const __attribute__((address_space(1))) V* global_ptr(const V* q) {
  return (const __attribute__((address_space(1))) V*)q;
}

// LDS of a list: CAP 16-bit entries and two rounds' counts per wave.
constexpr int list_bytes(int cap) { return cap * 2 + 2 * 16 * 4; }

// List the points from `pos` on for which keep(x, y) holds, in input order,
// as 16-bit offsets from pos, until the list may be full or the points end;
// returns their number and moves pos past the points tested.  Every thread of
// the workgroup (THREADS of them) calls it with the same arguments and gets
// the same result; it ends with a barrier.  One barrier per round of 2
// THREADS points: a wave's count of round k + 2 is written after the barrier
// of round k + 1, which every wave passes only after it has read the counts
// of round k.
template <int THREADS, int CAP, typename Keep>
__device__ __forceinline__ int list_points(const float* points, int64_t n, int64_t& pos,
                                           char* lds_list, Keep keep) {
  constexpr int kWaves = THREADS / 64, kScan = 2 * THREADS;
  static_assert(kScan <= CAP && kScan <= 65536 && kWaves <= 16, "list size");
  uint16_t* list = (uint16_t*)lds_list;
  int* counts = (int*)(lds_list + CAP * 2);   // [2][16]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t below = (1ull << lane) - 1ull;
  const int64_t base = pos;
  const auto pts = global_ptr(points);
  float x[2], y[2];
  auto load = [&](int64_t from) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t i = from + wave * 128 + q * 64 + lane;
      x[q] = i < n ? pts[2 * i] : 0.0f;
      y[q] = i < n ? pts[2 * i + 1] : 0.0f;
    }
  };
  int cnt = 0, buf = 0;
  load(pos);
  while (pos < n && pos - base <= 65536 - kScan) {
    const int64_t first = pos + wave * 128 + lane;
    const bool k0 = first < n && keep(x[0], y[0]);
    const bool k1 = first + 64 < n && keep(x[1], y[1]);
    load(pos + kScan);                     // the next round's, in flight
    const uint64_t m0 = __ballot(k0), m1 = __ballot(k1);
    const int c0 = __popcll(m0), c1 = __popcll(m1);
    if (lane == 0) counts[buf * 16 + wave] = c0 + c1;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int c = counts[buf * 16 + w];
      if (w < wave) before += c;
      total += c;
    }
    total = __builtin_amdgcn_readfirstlane(total);
    if (cnt + total > CAP) break;          // the same in every wave
    int o = cnt + before;
    if (k0) list[o + __popcll(m0 & below)] = (uint16_t)(first - base);
    o += c0;
    if (k1) list[o + __popcll(m1 & below)] = (uint16_t)(first + 64 - base);
    cnt += total;
    pos += kScan;
    buf ^= 1;
  }
  __syncthreads();
  return cnt;
}

}  // namespace mls
