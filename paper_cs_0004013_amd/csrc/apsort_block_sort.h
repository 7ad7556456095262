// Sort of up to WAVES * 64 * IPT keys held in the registers of one workgroup: the local radix sort
// of one cell (Weaver & Lynes, Sec. 3.3 / 3.3.1), with the workgroup as the cell.  Templates only.
//
// The keys are taken wave-striped (key j of lane l of wave w sits at w*64*IPT + j*64 + l), and each
// digit pass ranks them against the wave's own LDS counters, turns the counters into tile
// positions, and reorders the keys through LDS.  What bounds it is LDS latency and throughput, not
// memory: a pass is a chain of dependent LDS round trips and barriers, so
//   - digits are 8-bit windows laid over the bits that vary in the tile (diff), lowest first: bits
//     that every key shares cost nothing, and no pass runs for a digit before it is known to vary;
//   - a wave clears and reads only its own counters, so clearing needs no barrier;
//   - up to 4 waves, every wave sums all waves' counters by itself (WAVES 16-byte reads per lane)
//     and scans them with DPP moves: two barriers per pass.  With more waves those reads would
//     outweigh the barriers they save, and the counters are scanned once by the whole workgroup.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apsort_device.h"

namespace aps {

// Ranks of the workgroup sorts: SEG_RANK_ATOMIC with lane-ordered LDS atomics (rank_slot), selected
// by the host only on a device that passed the lane-order check; SEG_RANK_BALLOT with one ballot
// per digit bit (rank_ballot), which needs no ordering property of the LDS.
enum SegRank : int { SEG_RANK_ATOMIC = 0, SEG_RANK_BALLOT = 1 };

constexpr int kBlockBits = 8;
constexpr int kBlockRadix = 1 << kBlockBits;

// LDS of block_sort.  stage: WAVES*64*IPT words (vstage the same, with values); cnt: WAVES*256; off:
// WAVES*256 (2 to 4 waves only); scan: WAVES words.
struct BlockSortLds {
  uint32_t* stage;
  uint32_t* cnt;
  uint32_t* off;
  uint32_t* scan;
  uint32_t* vstage;
};

// Index of thread tid's first key in the tile.  With one wave the tile belongs to the wave, whatever
// its place in the workgroup.  (tid: threadIdx.x, in a loop over tiles fresh_tid().)
template <int WAVES, int IPT>
__device__ __forceinline__ uint32_t block_first(uint32_t tid) {
  return WAVES == 1 ? tid & 63u : (tid >> 6) * (64u * IPT) + (tid & 63u);
}

// A tile of len <= WAVES * 64 * IPT keys between memory and registers; the registers behind the
// last key get all-ones sentinels, which sort behind every key.
template <int WAVES, int IPT>
__device__ __forceinline__ void block_load(gptr<const uint32_t> in, uint32_t len, uint32_t (&k)[IPT],
                                           uint32_t tid = threadIdx.x) {
  const uint32_t lb0 = block_first<WAVES, IPT>(tid);
#pragma unroll
  for (int j = 0; j < IPT; ++j) k[j] = lb0 + j * 64u < len ? in[lb0 + j * 64u] : 0xFFFFFFFFu;
}

template <int WAVES, int IPT>
__device__ __forceinline__ void block_store(gptr<uint32_t> out, uint32_t len, const uint32_t (&k)[IPT],
                                            uint32_t tid = threadIdx.x) {
  const uint32_t lb0 = block_first<WAVES, IPT>(tid);
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    if (lb0 + j * 64u < len) out[lb0 + j * 64u] = k[j];
}

// Bits in which the tile's keys differ from the key `first`, ORed over the workgroup; uniform.
// scratch: WAVES words.  Contains one barrier (none with one wave).
template <int WAVES, int IPT>
__device__ __forceinline__ uint32_t varying_bits(const uint32_t (&k)[IPT], uint32_t first, uint32_t len,
                                                 uint32_t* scratch, uint32_t tid = threadIdx.x) {
  const uint32_t lb0 = block_first<WAVES, IPT>(tid);
  uint32_t x = 0u;
#pragma unroll
  for (int j = 0; j < IPT; ++j) x |= lb0 + j * 64u < len ? (k[j] ^ first) : 0u;
  x = wave_or(x);
  if constexpr (WAVES == 1) return x;
  if ((tid & 63u) == 0u) scratch[tid >> 6] = x;
  __syncthreads();
  x = 0u;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) x |= scratch[w];
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// Sorts the tile in k[] (sentinels all-ones behind the keys) on the bits set in diff: on return k[]
// holds the sorted tile in the same striped order, and so does the stage if diff was not zero.  Bits
// outside diff must be equal in all keys.  KV: the values in v[] move with their keys, equal keys
// keeping their order.
template <int WAVES, int IPT, int RANK, bool KV>
__device__ __forceinline__ void block_sort_impl(const BlockSortLds& sm, uint32_t (&k)[IPT], uint32_t* v,
                                                uint32_t diff, uint32_t tid = threadIdx.x) {
  constexpr int R = kBlockRadix;
  const int lane = (int)(tid & 63u), wid = WAVES == 1 ? 0 : (int)(tid >> 6);
  const uint32_t lb0 = block_first<WAVES, IPT>(tid);
  uint32_t* const cnt = sm.cnt + wid * R;
  uint32_t* const off = WAVES > 1 && WAVES <= 4 ? sm.off + wid * R : cnt;
  uint4* const cnt4 = reinterpret_cast<uint4*>(cnt);
  uint32_t r[IPT];
#pragma unroll 1
  while (diff) {
    const int shift = __builtin_ctz(diff);
    diff &= ~((uint32_t)(R - 1) << shift);
    cnt4[lane] = make_uint4(0u, 0u, 0u, 0u);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const uint32_t b = (k[j] >> shift) & (R - 1);
      if constexpr (RANK == SEG_RANK_ATOMIC) r[j] = rank_slot(cnt, b);
      else r[j] = rank_ballot<kBlockBits>(cnt, b);
    }
    if constexpr (WAVES <= 4) {
      // lane l of every wave takes buckets 4l .. 4l+3: their totals over the waves, their keys in
      // lower waves, and the scan of the totals
      if constexpr (WAVES > 1) __syncthreads();
      else __builtin_amdgcn_wave_barrier();
      uint4 tot = make_uint4(0u, 0u, 0u, 0u), low = tot;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const uint4 c = reinterpret_cast<const uint4*>(sm.cnt + w * R)[lane];
        if (w < wid) { low.x += c.x; low.y += c.y; low.z += c.z; low.w += c.w; }
        tot.x += c.x; tot.y += c.y; tot.z += c.z; tot.w += c.w;
      }
      const uint32_t s = tot.x + tot.y + tot.z + tot.w;
      const uint32_t b0 = wave_incl_scan(s) - s;
      const uint32_t b1 = b0 + tot.x, b2 = b1 + tot.y, b3 = b2 + tot.z;
      reinterpret_cast<uint4*>(off)[lane] = make_uint4(b0 + low.x, b1 + low.y, b2 + low.z, b3 + low.w);
      __builtin_amdgcn_wave_barrier();
    } else {
      tile_bucket_offsets<R, WAVES>(sm.cnt, nullptr, sm.scan, (int)tid);
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const uint32_t p = off[(k[j] >> shift) & (R - 1)] + r[j];
      sm.stage[p] = k[j];
      if constexpr (KV) sm.vstage[p] = v[j];
    }
    if constexpr (WAVES > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      k[j] = sm.stage[lb0 + j * 64u];
      if constexpr (KV) v[j] = sm.vstage[lb0 + j * 64u];
    }
  }
}

template <int WAVES, int IPT, int RANK>
__device__ __forceinline__ void block_sort(const BlockSortLds& sm, uint32_t (&k)[IPT], uint32_t diff,
                                           uint32_t tid = threadIdx.x) {
  block_sort_impl<WAVES, IPT, RANK, false>(sm, k, nullptr, diff, tid);
}

}  // namespace aps
