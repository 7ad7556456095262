// Sort of a short array by several workgroups in one launch, without a word exchanged between them:
// every workgroup reads the whole array (it fits one workgroup's registers), finds by counting which
// keys belong to its share of the ranks, sorts those alone and writes them to their place.
//
// For arrays of 4K to 16K keys: one workgroup is bound by the LDS of its one CU (16384 keys: 17.7 us,
// four digits of 256 rank and reorder steps each), two launches (apsort_cells.h) by their latencies
// (14 us); this takes 11 (uniform; 17 log-normal or in narrow bands, where the ends are found in three
// or four counts instead of one), and 8.5 to 9 for 4097 to 8192 keys where one workgroup takes 10.3.
// Reading the array once per workgroup costs little, it comes from the caches.  Not in place: a
// workgroup writes while others still read.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apsort_block_sort.h"
#include "apsort_device.h"

namespace aps {

// An end of a share while it is looked for: the rank lies in the bucket [value, value + last] of
// keys, with `below` keys under it, to be counted in steps of 2^shift; shift < 0: the share ends
// before `value`, with `below` keys under it.  (Past the largest key, value may wrap to 0.)
struct RankEnd {
  uint32_t value, last, below;
  int shift;
};

// Narrows an end by the counts h[256] of its bucket's steps: to the first step boundary at or above
// the rank, or, if the step that straddles the rank holds more than `fine` keys, into that step.
// Every wave computes it by itself.
__device__ __forceinline__ void rank_narrow(RankEnd& e, const uint32_t* h, uint32_t rank, uint32_t fine) {
  const uint4 c = reinterpret_cast<const uint4*>(h)[threadIdx.x & 63u];
  const uint32_t p1 = c.x, p2 = p1 + c.y, p3 = p2 + c.z, p4 = p3 + c.w;
  const uint32_t b = e.below + wave_incl_scan(p4) - p4;  // keys below this lane's first step
  // steps that start below the rank: a prefix of the 256, at least the first
  const uint32_t n = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(b < rank)) +
                     (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(b + p1 < rank)) +
                     (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(b + p2 < rank)) +
                     (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(b + p3 < rank));
  const uint32_t s = n - 1u, q = s & 3u;  // the last of them
  const uint32_t at = q == 0u ? b : q == 1u ? b + p1 : q == 2u ? b + p2 : b + p3;
  const uint32_t start = (uint32_t)__builtin_amdgcn_readlane((int)at, (int)(s >> 2));
  const uint32_t held = q == 0u ? c.x : q == 1u ? c.y : q == 2u ? c.z : c.w;
  const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)held, (int)(s >> 2));
  if (cnt > fine && e.shift > 0) {
    e.value += s << e.shift;
    e.last = (1u << e.shift) - 1u;
    e.below = start;
    e.shift = max(e.shift - 8, 0);
  } else {
    e.value += (uint32_t)((uint64_t)n << e.shift);
    e.below = start + cnt;
    e.shift = -1;
  }
}

// Sorts the stage's cnt <= 512 * IPT keys (8 waves) and writes them to out[0..cnt).  Returns the bits
// sorted on; if there are none every key is `first`, else the sorted keys are in the stage too.
template <int IPT, int RANK, int I = IPT>
__device__ __forceinline__ uint32_t rank_share_sort(const BlockSortLds& lds, gptr<uint32_t> out, uint32_t cnt, uint32_t& first) {
  if constexpr (I > 1) {
    constexpr int S = I == 8 ? 6 : I == 6 ? 4 : I == 4 ? 3 : I == 3 ? 2 : I / 2;
    if (cnt <= 512u * S) return rank_share_sort<IPT, RANK, S>(lds, out, cnt, first);
  }
  const uint32_t lb0 = block_first<8, I>(threadIdx.x);
  uint32_t k[I];
#pragma unroll
  for (int j = 0; j < I; ++j) k[j] = lb0 + j * 64u < cnt ? lds.stage[lb0 + j * 64u] : 0xFFFFFFFFu;
  first = lds.stage[0];
  const uint32_t diff = varying_bits<8, I>(k, first, cnt, lds.scan);
  block_sort<8, I, RANK>(lds, k, diff);
  block_store<8, I>(out, cnt, k);
  return diff;
}

template <int IPT, int RANK>
__global__ __launch_bounds__(512) void k_sort_ranks(const uint32_t* __restrict__ in, uint32_t* __restrict__ out, uint32_t n,
                                                   uint32_t P, uint32_t* __restrict__ spl) {
  constexpr uint32_t THREADS = 512, WAVES = 8;
  // Counts in 8 copies, a lane adding to copy lane % 8: keys that crowd into few steps (narrow bands, a
  // long tail) would queue on one word lane by lane (12345 log-normal keys: 31 us with one copy).
  constexpr uint32_t COPIES = 8, CS = 257;
  static_assert(2u * COPIES * CS <= THREADS * IPT, "the counts share the stage");
  __shared__ __align__(16) uint32_t s_stage[THREADS * IPT];
  __shared__ __align__(16) uint32_t s_cnt[WAVES * kBlockRadix];
  __shared__ __align__(16) uint32_t s_hist[2][256];
  __shared__ uint32_t s_scan[WAVES];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6, g = blockIdx.x, G = gridDim.x;
  const BlockSortLds lds{s_stage, s_cnt, nullptr, s_scan, nullptr};
  const uint32_t lb0 = block_first<WAVES, IPT>(tid);
  uint32_t k[IPT];
  block_load<WAVES, IPT>(gmem(in), n, k);
  const uint32_t first = in[0];
  const uint32_t diff = varying_bits<WAVES, IPT>(k, first, n, s_scan);
  // ranks [g*n/G, (g+1)*n/G), n <= 2^14 and G <= 2^6
  const uint32_t rank_a = g * n / G, rank_b = (g + 1u) * n / G, fine = n / G;
  RankEnd a{0u, 0u, 0u, -1}, b{0u, 0u, n, -1};
  if (diff) {
    const uint32_t mask = 0xFFFFFFFFu >> __builtin_clz(diff);  // the highest varying bit and all below
    const RankEnd whole{first & ~mask, mask, 0u, max(24 - __builtin_clz(diff), 0)};
    if (g > 0u) a = whole;
    if (g + 1u < G) b = whole;
    while (a.shift >= 0 || b.shift >= 0) {  // uniform over the workgroup
      const bool one = a.shift >= 0 && b.shift >= 0 && a.value == b.value && a.last == b.last;
      for (uint32_t i = tid; i < (one ? 1u : 2u) * COPIES * CS; i += THREADS) s_stage[i] = 0u;
      __syncthreads();
      uint32_t* const ha = s_stage + (lane % COPIES) * CS;
      uint32_t* const hb = ha + COPIES * CS;
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        if (lb0 + j * 64u < n) {
          if (a.shift >= 0 && k[j] - a.value <= a.last) atomicAdd(&ha[(k[j] - a.value) >> a.shift], 1u);
          if (b.shift >= 0 && !one && k[j] - b.value <= b.last) atomicAdd(&hb[(k[j] - b.value) >> b.shift], 1u);
        }
      }
      __syncthreads();
      if (!one || tid < 256u) {
        const uint32_t* const h = s_stage + (tid >> 8) * COPIES * CS + (tid & 255u);
        uint32_t c = 0u;
#pragma unroll
        for (uint32_t i = 0; i < COPIES; ++i) c += h[i * CS];
        s_hist[tid >> 8][tid & 255u] = c;
      }
      __syncthreads();
      if (b.shift >= 0) rank_narrow(b, s_hist[one ? 0 : 1], rank_b, fine);  // one: the same bucket for both
      if (a.shift >= 0) rank_narrow(a, s_hist[0], rank_a, fine);
    }
  } else {  // one value: any share of the ranks will do
    a.below = rank_a;
    b.below = rank_b;
  }
  const uint32_t base = a.below, cnt = b.below - a.below;
  if (cnt == 0u) return;
  uint32_t value = first, bits = 0u;
  if (diff) {
    // the share's keys, in any order: each wave's after the lower waves', each lane's after the lower
    // lanes' (an end at 0 is no end: the first share starts, the last one ends there)
    uint32_t mine = 0u;
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      mine += lb0 + j * 64u < n && k[j] >= a.value && k[j] <= b.value - 1u ? 1u : 0u;
    const uint32_t ic = wave_incl_scan(mine);
    if (lane == 63u) s_scan[wid] = ic;
    __syncthreads();
    uint32_t p = ic - mine;
#pragma unroll
    for (uint32_t w = 0; w < WAVES; ++w) p += w < wid ? s_scan[w] : 0u;
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      if (lb0 + j * 64u < n && k[j] >= a.value && k[j] <= b.value - 1u) s_stage[p++] = k[j];
    __syncthreads();
    bits = rank_share_sort<IPT, RANK>(lds, gmem(out) + base, cnt, value);
  } else {
    for (uint32_t i = tid; i < cnt; i += THREADS) out[base + i] = first;
  }
  if (!spl) return;
  const uint32_t q = n / P, r = n % P;
  for (uint32_t c = tid + 1u; c < P; c += THREADS) {
    const uint64_t at = (uint64_t)c * q + min(c, r);
    if (at >= base && at < base + cnt) spl[c - 1u] = bits ? s_stage[at - base] : value;
    else if (at >= n && base + cnt == n) spl[c - 1u] = 0xFFFFFFFFu;
  }
}

}  // namespace aps
