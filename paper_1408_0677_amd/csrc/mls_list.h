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

// The lists are in LDS, said as explicitly.
typedef __attribute__((address_space(3))) char* LdsBytes;

// LDS of a list: CAP 16-bit entries (the masks they are made from before) and
// two sets of per-wave values.
constexpr int list_bytes(int cap) { return cap * 2 + 2 * 16 * 4; }

// A value that is the same in every lane, in scalar registers.
template <typename V>
__device__ __forceinline__ V uniform(V v) {
  static_assert(sizeof(V) % 4 == 0, "whole registers");
  struct Words {
    int w[sizeof(V) / 4];
  };
  Words u = __builtin_bit_cast(Words, v);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(V) / 4); ++i) u.w[i] = __builtin_amdgcn_readfirstlane(u.w[i]);
  return __builtin_bit_cast(V, u);
}

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
  return v;
}

// List the points from `pos` on for which keep(x, y) holds, in input order,
// as 16-bit offsets from pos, until the list would be full or a window of 16
// CAP points ends; returns their number and moves pos past the points taken.
// Every thread of the workgroup (THREADS of them) calls it with the same
// arguments and gets the same result; it ends with a barrier.
//
// The tests bound it (every tile of a call looks at every point; 50,000 points
// took a tile of the bfloat16 fit 87,000 cycles in rounds that each counted,
// met at a barrier and wrote their entries, and take 42,000), so a wave does
// no more than that for a group of 64 points: its 64-bit mask goes to a
// lane of a register pair and to LDS with the wave's other masks, without a
// word to the other waves, and the next groups' points are loaded meanwhile
// from a scalar address.  The last group ends with the last point, so it
// repeats points of the group before; their bits are cleared when the masks
// are read, by consecutive threads, counted and unpacked into the space that
// they leave.  keep may see a point more than once and must not depend on it.
template <int THREADS, int CAP, typename Keep>
__device__ __forceinline__ int list_points(const float* points, int64_t n, int64_t& pos,
                                           LdsBytes lds_list, Keep keep) {
  constexpr int kWaves = THREADS / 64, kWindow = 16 * CAP, U = 4;
  constexpr int kPer = (kWindow / 16 + THREADS - 1) / THREADS;
  static_assert(kWindow <= 65536 && CAP >= 64 && kWaves <= 16, "list size");
  const auto masks = (__attribute__((address_space(3))) uint64_t*)lds_list;
  const auto list = (__attribute__((address_space(3))) uint16_t*)lds_list;
  const auto counts = (__attribute__((address_space(3))) int*)(lds_list + CAP * 2);   // per wave; [16], [17]: a cut
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lim = (int)(n - pos < kWindow ? n - pos : kWindow);
  if (lim <= 0) return 0;
  const int groups = (lim + 63) >> 6;
  const int last = lim > 64 ? lim - 64 : 0;   // the last group's first point
  const auto pts = global_ptr((const char*)points) + 8 * pos;
  const uint32_t vo = 8u * (uint32_t)min(lane, lim - 1);
  auto load = [&](int g, float (&x)[U], float (&y)[U]) {
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const auto pt = (const __attribute__((address_space(1))) float*)(
          pts + (uint32_t)(8 * min((g + q * kWaves) * 64, last)) + vo);
      x[q] = pt[0];
      y[q] = pt[1];
    }
  };
  uint32_t lo = 0, hi = 0;   // lane k: the wave's k-th mask since `done`
  int k = 0, done = wave;
  auto flush = [&]() {
    if (lane < k) masks[done + lane * kWaves] = (uint64_t)hi << 32 | lo;
    done += k * kWaves;
    k = 0;
  };
  auto test = [&](int g, const float (&x)[U], const float (&y)[U]) {
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const uint64_t m = __builtin_amdgcn_ballot_w64(keep(x[q], y[q]));
      if (g + q * kWaves < groups) {
        lo = lane == k ? (uint32_t)m : lo;
        hi = lane == k ? (uint32_t)(m >> 32) : hi;
        ++k;
      }
    }
    if (k > 64 - U) flush();
  };
  {
    float xa[U], ya[U], xb[U], yb[U];
    int g = wave;
    load(g, xa, ya);
    while (g < groups) {
      load(g + U * kWaves, xb, yb);
      test(g, xa, ya);
      g += U * kWaves;
      if (g >= groups) break;
      load(g + U * kWaves, xa, ya);
      test(g, xb, yb);
      g += U * kWaves;
    }
    flush();
  }
  __syncthreads();
  // unpacked by 16 bits, which keeps the threads' shares even where most
  // points are listed
  const auto bits = (__attribute__((address_space(3))) uint16_t*)lds_list;
  const int pieces = 4 * groups;
  const int per = (pieces + THREADS - 1) / THREADS;   // a thread's, <= kPer
  uint32_t b[kPer];
  int c = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = tid * per + q;
    b[q] = q < per && e < pieces ? bits[e] : 0;
    if (e >= pieces - 4) {
      const uint64_t valid = lim < 64 ? (1ull << lim) - 1 : ~0ull << (64 * groups - lim);
      b[q] &= (uint32_t)(valid >> (16 * (e & 3)));
    }
    c += __builtin_popcount(b[q]);
  }
  const int incl = wave_scan(c);
  if (lane == 63) counts[wave] = incl;
  __syncthreads();
  int o = incl - c, cnt = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int cw = counts[w];
    if (w < wave) o += cw;
    cnt += cw;
  }
  cnt = __builtin_amdgcn_readfirstlane(cnt);
  auto first = [&](int e) { return min((e >> 2) * 64, last) + 16 * (e & 3); };
  int taken = lim;
  if (cnt > CAP) {
    // the first piece that would not fit ends the list
    int at = o;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = tid * per + q, next = at + __builtin_popcount(b[q]);
      if (at <= CAP && next > CAP) {
        counts[16] = at;
        counts[17] = max(first(e), (e >> 2) * 64);
      }
      if (next > CAP) b[q] = 0;
      at = next;
    }
    __syncthreads();
    cnt = __builtin_amdgcn_readfirstlane(counts[16]);
    taken = __builtin_amdgcn_readfirstlane(counts[17]);
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int f = first(tid * per + q);
    while (b[q]) {
      list[o++] = (uint16_t)(f + __builtin_ctz(b[q]));
      b[q] &= b[q] - 1;
    }
  }
  pos += taken;
  __syncthreads();
  return cnt;
}

// Drop the entries of a list (from point `base`, cnt of them) for which
// keep(x, y, sum) does not hold; returns how many are left.  `sum` is that of
// add(x, y) over the list (the same bits in every thread, and for the same
// list in every kernel).  Called and synchronised as list_points; a
// wave's entries are consecutive, and all are read before any is written.
template <int THREADS, int CAP, typename Add, typename Keep>
__device__ __forceinline__ int refine_list(const float* points, int64_t base, int cnt,
                                           LdsBytes lds_list, Add add, Keep keep) {
  constexpr int kWaves = THREADS / 64, PT = (CAP + THREADS - 1) / THREADS;
  if (cnt == 0) return 0;
  const auto list = (__attribute__((address_space(3))) uint16_t*)lds_list;
  const auto counts = (__attribute__((address_space(3))) int*)(lds_list + CAP * 2);
  const auto sums = (__attribute__((address_space(3))) float*)(lds_list + CAP * 2) + 16;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t below = (1ull << lane) - 1ull;
  const auto pts = global_ptr(points) + 2 * base;
  const int per = __builtin_amdgcn_readfirstlane((cnt + THREADS - 1) / THREADS);
  const int first = wave * per * 64 + lane;
  uint16_t v[PT];
  float x[PT], y[PT];
#pragma unroll
  for (int q = 0; q < PT; ++q) {
    v[q] = 0;
    x[q] = y[q] = 0.0f;
    if (q < per) {
      v[q] = list[min(first + q * 64, cnt - 1)];
      x[q] = pts[2 * (int)v[q]];
      y[q] = pts[2 * (int)v[q] + 1];
    }
  }
  float sum = 0.0f;
#pragma unroll
  for (int q = 0; q < PT; ++q)
    if (q < per) sum += first + q * 64 < cnt ? add(x[q], y[q]) : 0.0f;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (lane == 0) sums[wave] = sum;
  __syncthreads();
  sum = 0.0f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) sum += sums[w];
  sum = uniform(sum);
  uint64_t m[PT];
  int c = 0;
#pragma unroll
  for (int q = 0; q < PT; ++q) {
    m[q] = q < per ? __ballot((first + q * 64 < cnt) & keep(x[q], y[q], sum)) : 0;
    c += __popcll(m[q]);
  }
  if (lane == 0) counts[wave] = c;
  __syncthreads();
  int o = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int cw = counts[w];
    if (w < wave) o += cw;
    total += cw;
  }
#pragma unroll
  for (int q = 0; q < PT; ++q) {
    if (m[q] >> lane & 1) list[o + __popcll(m[q] & below)] = v[q];
    o += __popcll(m[q]);
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(total);
}

}  // namespace mls
