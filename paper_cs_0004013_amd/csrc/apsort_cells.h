// Sort of an array in two launches: split it into cells of neighbouring keys, then sort every cell
// in one workgroup (Weaver & Lynes, Sec. 3.2: distribution of the keys into ranges, then the local
// sort of Sec. 3.3 in each cell).  Templates only.
//
//   k_split  one workgroup per tile of the input: draws a sample of the whole array (the same one in
//            every workgroup), sorts it, takes every (M/B)-th key of it as a splitter, ranks the
//            tile's keys by cell, and writes the tile back ordered by cell, with the tile's cell
//            starts in one row of a table.  Nothing is communicated between workgroups.
//   k_cells  one workgroup per cell: sums the column of the table before it (the cell's place in
//            the output), gathers the cell's pieces from all tiles, sorts them (block_sort) and
//            writes them out, with the splitters of the output contract that fall into it.
//
// What it is for: arrays too long for one workgroup and too short to fill the device, where the
// digit passes are bound by their launches and look-back chains: six launches that each wait for
// the one before.  Here two launches move 16 B per key, and no workgroup waits for another.
//
// Cell of a key: the number of splitters below it.  Equal sample keys make equal splitters s[i] =
// s[i+1] = ..., between which no key could lie; a key equal to such a splitter goes to cell i+1, so
// that a value holding more than a cell's share of the array gets a cell of its own, in which
// nothing needs sorting.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apsort_block_sort.h"
#include "apsort_device.h"

namespace aps {

constexpr int kLutBits = 11;  // key prefixes of the cell look-up table
constexpr int kLutSize = 1 << kLutBits;

// Position i (of m) of the sample of n >= m keys: one key out of every n / m, at a scrambled place
// of its stretch, so that a period in the input does not show in the sample.
__device__ __forceinline__ uint32_t sample_pos(uint32_t i, uint32_t stride) {
  uint32_t h = i * 0x9E3779B9u;
  h ^= h >> 15;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  return i * stride + __umulhi(h, stride);
}

// Sorts M = WAVES*64*SI sample keys of in[0..n) in LDS and leaves B-1 splitters in spl[0..B-1), with
// all-ones behind them up to 2B.  Ends with a barrier.
// The sample is first sorted on its 16 highest varying bits alone, the lower ones cleared: two digit
// passes instead of four.  Splitters made of those bits are as good as long as no two of them are
// equal; if some are (narrow bands of keys, or a value that fills more than a cell), the whole keys
// are sorted.
template <int WAVES, int SI, int B, int RANK>
__device__ __forceinline__ void split_sample(const BlockSortLds& lds, gptr<const uint32_t> in, uint32_t n, uint32_t* spl) {
  constexpr int THREADS = WAVES * 64, M = THREADS * SI;
  static_assert(M % B == 0, "whole sample steps per cell");
  static_assert(WAVES > 4, "the tile sort of up to 4 waves needs position words of its own");
  const int tid = threadIdx.x, wid = tid >> 6, lane = tid & 63;
  const uint32_t stride = n / (uint32_t)M;
  uint32_t ks[SI];
#pragma unroll
  for (int j = 0; j < SI; ++j) ks[j] = in[sample_pos((uint32_t)(wid * 64 * SI + j * 64 + lane), stride)];
  const uint32_t first = in[sample_pos(0u, stride)];
  const uint32_t diff = varying_bits<WAVES, SI>(ks, first, (uint32_t)M, lds.scan);
  const uint32_t low = diff >> 16 ? (1u << (16 - __builtin_clz(diff))) - 1u : 0u;  // below the 16 highest
#pragma unroll 1
  for (uint32_t part = low ? diff & ~low : diff;; part = diff) {
    const uint32_t drop = part == diff ? 0u : low;
    block_sort<WAVES, SI, RANK>(lds, ks, part);
    for (int j = tid; j < 2 * B; j += THREADS)
      spl[j] = j < B - 1 ? (part ? lds.stage[(j + 1) * (M / B)] : first) & ~drop : 0xFFFFFFFFu;
    __syncthreads();
    if (!drop) return;
    bool eq = false;
    for (int j = tid; j + 1 < B - 1; j += THREADS) eq |= spl[j] == spl[j + 1];
    if (!__syncthreads_or(eq)) return;
  }
}

// Cell look-up: lut[p] = number of splitters below the start of prefix p of the range
// [spl[0], spl[B-2]]; a key's cell is lut[its prefix] plus the splitters of the prefix below the
// key, found by `steps` halvings (2^steps exceeds the splitters of any prefix).
struct CellMap {
  uint32_t s0, shift;
  int steps;   // uniform
  bool equal;  // some neighbouring splitters are equal
};

template <int WAVES, int B>
__device__ __forceinline__ CellMap split_map(const uint32_t* spl, uint16_t* lut, uint32_t* scratch) {
  constexpr int THREADS = WAVES * 64;
  const int tid = threadIdx.x;
  CellMap m;
  m.s0 = spl[0];
  const uint32_t range = spl[B - 2] - m.s0;
  m.shift = range >> kLutBits ? (uint32_t)(32 - kLutBits) - (uint32_t)__clz((int)range) : 0u;
  if (tid == 0) scratch[0] = scratch[1] = 0u;
#pragma unroll
  for (int q = 0; q < (kLutSize + THREADS - 1) / THREADS; ++q) {
    const int p = q * THREADS + tid;
    // splitters below the prefix's start (saturated: a prefix past the last splitter has them all)
    const uint64_t at = (uint64_t)m.s0 + ((uint64_t)p << m.shift);
    const uint32_t key = at > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)at;
    uint32_t c = 0;
#pragma unroll
    for (int s = B / 2; s > 0; s >>= 1)
      if (spl[c + s - 1] < key) c += s;
    if (p < kLutSize) lut[p] = (uint16_t)c;
  }
  __syncthreads();
  uint32_t most = 0u, eq = 0u;
  for (int p = tid; p < kLutSize; p += THREADS)
    most = max(most, (p + 1 < kLutSize ? (uint32_t)lut[p + 1] : (uint32_t)(B - 1)) - lut[p]);
  for (int j = tid; j + 1 < B - 1; j += THREADS) eq |= spl[j] == spl[j + 1] ? 1u : 0u;
  atomicMax(&scratch[0], most);
  if (eq) scratch[1] = 1u;
  __syncthreads();
  most = (uint32_t)__builtin_amdgcn_readfirstlane((int)scratch[0]);
  m.equal = __builtin_amdgcn_readfirstlane((int)scratch[1]) != 0;
  m.steps = most ? 32 - __clz((int)most) : 0;
  return m;
}

// One tile of the array ordered by cell.  tmp, table and splitters are written; in the table a tile
// has one row of B cell starts.
// A chain of LDS round trips and barriers (sample sort, look-up table, ranks, scan), 9-15 us for a
// tile however large the array, so long as its tiles fit the device at once; memory is idle most of
// that time.
template <int WAVES, int IPT, int SI, int B, int RANK, bool KV>
__global__ __launch_bounds__(WAVES * 64) void k_split(const uint32_t* __restrict__ in, const uint32_t* __restrict__ vin,
                                                     uint32_t* __restrict__ tmp, uint32_t* __restrict__ vtmp,
                                                     uint32_t n, uint16_t* __restrict__ table,
                                                     uint32_t* __restrict__ splitters) {
  constexpr int THREADS = WAVES * 64, T = THREADS * IPT;
  constexpr int CW = B > kBlockRadix ? B : kBlockRadix;
  __shared__ __align__(16) uint32_t s_stage[T];
  __shared__ __align__(16) uint32_t s_vstage[KV ? T : 4];
  __shared__ __align__(16) uint32_t s_cnt[WAVES * CW];
  __shared__ uint32_t s_spl[2 * B];
  __shared__ uint16_t s_lut[kLutSize];
  __shared__ uint32_t s_lbase[B + 1];
  __shared__ uint32_t s_scan[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint32_t tbase = blockIdx.x * (uint32_t)T;
  const uint32_t len = min(n - tbase, (uint32_t)T);
  const gptr<const uint32_t> gin = gmem(in);
  const BlockSortLds lds{s_stage, s_cnt, nullptr, s_scan, nullptr};
  split_sample<WAVES, SI, B, RANK>(lds, gin, n, s_spl);
  if (blockIdx.x == 0)
    for (int j = tid; j < B - 1; j += THREADS) splitters[j] = s_spl[j];
  uint32_t k[IPT], v[KV ? IPT : 1];
  block_load<WAVES, IPT>(gin + tbase, len, k);
  if constexpr (KV) block_load<WAVES, IPT>(gmem(vin) + tbase, len, v);
  const CellMap m = split_map<WAVES, B>(s_spl, s_lut, s_scan);
  uint32_t id[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) id[j] = s_lut[min((max(k[j], m.s0) - m.s0) >> m.shift, (uint32_t)(kLutSize - 1))];
  for (int st = m.steps - 1; st >= 0; --st) {
    const uint32_t step = 1u << st;
#pragma unroll
    for (int j = 0; j < IPT; ++j) id[j] += s_spl[id[j] + step - 1u] < k[j] ? step : 0u;
  }
  if (m.equal) {
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      if (id[j] + 1u < (uint32_t)(B - 1) && s_spl[id[j]] == k[j] && s_spl[id[j] + 1u] == k[j]) ++id[j];
  }
  for (int i = tid; i < WAVES * B; i += THREADS) s_cnt[i] = 0u;
  __syncthreads();
  uint32_t* const cnt = s_cnt + wid * B;
  uint32_t r[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    if constexpr (RANK == SEG_RANK_ATOMIC) r[j] = rank_slot(cnt, id[j]);
    else r[j] = rank_ballot<__builtin_ctz(B)>(cnt, id[j]);
  }
  tile_bucket_offsets<B, WAVES>(s_cnt, s_lbase, s_scan);
  for (int b = tid; b < B; b += THREADS) table[(size_t)blockIdx.x * B + b] = (uint16_t)min(s_lbase[b], len);
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const uint32_t p = cnt[id[j]] + r[j];
    s_stage[p] = k[j];
    if constexpr (KV) s_vstage[p] = v[j];
  }
  __syncthreads();
  const gptr<uint32_t> out = gmem(tmp) + tbase, vout = gmem(vtmp) + (KV ? tbase : 0u);
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const uint32_t i = (uint32_t)(j * THREADS + tid);
    if (i < len) {
      out[i] = s_stage[i];
      if constexpr (KV) vout[i] = s_vstage[i];
    }
  }
}

// Pairs short enough for one workgroup: the tile sort alone, in one launch.
template <int WAVES, int IPT, int RANK, int I = IPT>
__device__ __forceinline__ void sort_pairs_tile(const BlockSortLds& lds, const uint32_t* kin, const uint32_t* vin, uint32_t* kout,
                                                uint32_t* vout, uint32_t n, uint32_t P, uint32_t* spl) {
  if constexpr (I > 1) {
    if (n <= (uint32_t)(WAVES * 64 * (I / 2))) {
      sort_pairs_tile<WAVES, IPT, RANK, I / 2>(lds, kin, vin, kout, vout, n, P, spl);
      return;
    }
  }
  uint32_t k[I], v[I];
  block_load<WAVES, I>(gmem(kin), n, k);
  block_load<WAVES, I>(gmem(vin), n, v);
  const uint32_t first = kin[0];
  const uint32_t diff = varying_bits<WAVES, I>(k, first, n, lds.scan);
  block_sort_impl<WAVES, I, RANK, true>(lds, k, v, diff);
  block_store<WAVES, I>(gmem(kout), n, k);
  block_store<WAVES, I>(gmem(vout), n, v);
  if (!spl) return;
  const uint32_t q = n / P, r = n % P;
  for (uint32_t p = threadIdx.x + 1u; p < P; p += WAVES * 64) {
    const uint64_t at = (uint64_t)p * q + min(p, r);
    spl[p - 1u] = at < n ? (diff ? lds.stage[at] : first) : 0xFFFFFFFFu;
  }
}
template <int WAVES, int IPT, int RANK>
__global__ __launch_bounds__(WAVES * 64) void k_sort_pairs_small(const uint32_t* kin, const uint32_t* vin, uint32_t* kout,
                                                                uint32_t* vout, uint32_t n, uint32_t P, uint32_t* spl) {
  __shared__ __align__(16) uint32_t s_stage[WAVES * 64 * IPT], s_vstage[WAVES * 64 * IPT];
  __shared__ __align__(16) uint32_t s_cnt[WAVES * kBlockRadix], s_off[WAVES <= 4 ? WAVES * kBlockRadix : 4];
  __shared__ uint32_t s_scan[WAVES];
  const BlockSortLds lds{s_stage, s_cnt, s_off, s_scan, s_vstage};
  sort_pairs_tile<WAVES, IPT, RANK>(lds, kin, vin, kout, vout, n, P, spl);
}

// First cell p >= 0 of the output contract that starts at position x or later (P cells over n keys,
// the first n mod P of them one key longer).
__device__ __forceinline__ uint32_t first_cell_from(uint32_t x, uint32_t q, uint32_t r) {
  const uint32_t big = r * (q + 1u);  // keys in the longer cells; <= n
  return x <= big ? (x + q) / (q + 1u) : r + (x - big + q - 1u) / q;
}

struct CellsLds {
  BlockSortLds sort;
  uint32_t* poff;   // [THREADS] first position of each piece in the cell, all-ones past the last tile
  uint32_t* psrc;   // [THREADS] place of the piece in the split array minus poff
  uint32_t* scan2;  // [WAVES]
};

// A split array, as k_split left it.
struct SplitArray {
  const uint32_t* keys;
  const uint32_t* vals;
  const uint16_t* table;
  uint32_t n, ntiles, tile, ncells;
};

// Where position i of the cell lies in the split array: the piece is the last one that starts at or
// before i, found by halvings over the pieces' starts (lanes of neighbouring positions read the
// same words).
__device__ __forceinline__ uint32_t cell_src(const CellsLds& lds, uint32_t top, uint32_t i) {
  uint32_t t = 0u;
  for (uint32_t s = top; s > 0u; s >>= 1)
    if (lds.poff[t + s] <= i) t += s;
  return lds.psrc[t] + i;
}

// The pieces of cell b: poff and psrc from the table's columns b and b+1; returns the cell's length
// and its place in the sorted array (the keys of lower cells: the sum of the tile-local starts).
// At most THREADS tiles.  Ends with a barrier.
template <int WAVES>
__device__ __forceinline__ uint2 cell_pieces(const CellsLds& lds, const SplitArray& a, uint32_t b) {
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
  uint32_t start = 0u, cnt = 0u;
  if (tid < a.ntiles) {
    const uint16_t* const row = a.table + (size_t)tid * a.ncells + b;
    start = row[0];
    cnt = (b + 1u < a.ncells ? (uint32_t)row[1] : min(a.n - tid * a.tile, a.tile)) - start;
  }
  const uint32_t ic = wave_incl_scan(cnt), is = wave_incl_scan(start);
  __syncthreads();  // a previous cell's pieces are no longer read
  if (lane == 63u) {
    lds.sort.scan[wid] = ic;
    lds.scan2[wid] = is;
  }
  __syncthreads();
  uint32_t pre = 0u, len = 0u, base = 0u;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const uint32_t x = lds.sort.scan[w];
    pre += w < (int)wid ? x : 0u;
    len += x;
    base += lds.scan2[w];
  }
  const uint32_t off = pre + ic - cnt;
  lds.poff[tid] = tid < a.ntiles ? off : 0xFFFFFFFFu;
  lds.psrc[tid] = tid * a.tile + start - off;
  __syncthreads();
  return make_uint2((uint32_t)__builtin_amdgcn_readfirstlane((int)len), (uint32_t)__builtin_amdgcn_readfirstlane((int)base));
}

// Sorts a cell of len <= WAVES*64*IPT keys, none below lo, into out[0..len).  Keys per lane by
// length, in steps of 1.33 to 1.5.  Returns the bits sorted on (0: every key is lo).
template <int WAVES, int IPT, int RANK, bool KV, int I = IPT>
__device__ __forceinline__ uint32_t cell_sort_tile(const CellsLds& lds, const SplitArray& a, gptr<uint32_t> out,
                                                   gptr<uint32_t> vout, uint32_t top, uint32_t len, uint32_t lo) {
  static_assert(WAVES > 4, "the tile sort of up to 4 waves needs position words of its own");
  if constexpr (I > 1) {
    constexpr int S = I == 20 ? 16 : I == 16 ? 12 : I == 12 ? 8 : I == 8 ? 6 : I == 6 ? 4 : I / 2;
    if (len <= (uint32_t)(WAVES * 64 * S)) return cell_sort_tile<WAVES, IPT, RANK, KV, S>(lds, a, out, vout, top, len, lo);
  }
  const gptr<const uint32_t> keys = gmem(a.keys), vals = gmem(a.vals);
  const uint32_t lb0 = (threadIdx.x >> 6) * (64u * I) + (threadIdx.x & 63u);
  uint32_t k[I], v[KV ? I : 1], src[I];
#pragma unroll
  for (int j = 0; j < I; ++j) src[j] = 0u;
  // halvings of all the lane's positions together: their reads overlap
  for (uint32_t s = top; s > 0u; s >>= 1) {
#pragma unroll
    for (int j = 0; j < I; ++j) src[j] += lds.poff[src[j] + s] <= lb0 + j * 64u ? s : 0u;
  }
#pragma unroll
  for (int j = 0; j < I; ++j) src[j] = lds.psrc[src[j]] + lb0 + j * 64u;
#pragma unroll
  for (int j = 0; j < I; ++j) k[j] = lb0 + j * 64u < len ? keys[src[j]] - lo : 0xFFFFFFFFu;
  if constexpr (KV) {
#pragma unroll
    for (int j = 0; j < I; ++j) v[j] = lb0 + j * 64u < len ? vals[src[j]] : 0u;
  }
  const uint32_t diff = varying_bits<WAVES, I>(k, 0u, len, lds.sort.scan);
  block_sort_impl<WAVES, I, RANK, KV>(lds.sort, k, v, diff);
#pragma unroll
  for (int j = 0; j < I; ++j)
    if (lb0 + j * 64u < len) {
      out[lb0 + j * 64u] = k[j] + lo;
      if constexpr (KV) vout[lb0 + j * 64u] = v[j];
    }
  return diff;
}

// Writes positions [i0, i1) of a cell whose keys all equal `key`: the key itself and, with values,
// the cell's values in their order.
template <int THREADS, bool KV>
__device__ __forceinline__ void cell_fill(const CellsLds& lds, const SplitArray& a, gptr<uint32_t> out,
                                          gptr<uint32_t> vout, uint32_t top, uint32_t i0, uint32_t i1, uint32_t key) {
  const gptr<const uint32_t> vals = gmem(a.vals);
  if constexpr (!KV) {
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += THREADS) out[i] = key;
    return;
  }
  // four positions at a time: their searches and loads overlap
  for (uint32_t i = i0 + threadIdx.x; i < i1; i += 4u * THREADS) {
    uint32_t src[4], val[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) src[u] = 0u;
    for (uint32_t st = top; st > 0u; st >>= 1) {
#pragma unroll
      for (int u = 0; u < 4; ++u) src[u] += lds.poff[src[u] + st] <= i + u * THREADS ? st : 0u;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) val[u] = i + u * THREADS < i1 ? vals[lds.psrc[src[u]] + i + u * THREADS] : 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u * THREADS < i1) {
        out[i + u * THREADS] = key;
        vout[i + u * THREADS] = val[u];
      }
  }
}

// A cell longer than one tile whose keys differ (the sample missed the cell's keys): counted over 256
// equal steps of its key range [lo, lo + range), then sorted tile by tile, each tile the longest run
// of steps that fits, read out of the cell in its order; a step too long by itself is counted again
// over finer steps, down to single values.  The cell is read once per count and per tile, and needs
// no scratch: a cell of 10000 keys takes about 40 us.
template <int WAVES, int IPT, int RANK, bool KV>
__device__ __forceinline__ void cell_sort_oversize(const CellsLds& lds, const SplitArray& a, uint32_t* out_p, uint32_t* vout_p,
                                   uint32_t top, uint32_t len, uint32_t lo, uint64_t range) {
  constexpr uint32_t THREADS = WAVES * 64, CAP = THREADS * IPT;
  constexpr int U = 4;  // keys per thread and step: their searches and loads overlap
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
  const gptr<const uint32_t> keys = gmem(a.keys), vals = gmem(a.vals);
  const gptr<uint32_t> out = gmem(out_p), vout = gmem(vout_p);
  uint32_t* const h = lds.sort.cnt;         // 256 counts, [256] steps taken, [257] their keys
  uint32_t* const part = lds.sort.cnt + 512;  // [U * WAVES] keys found by each wave and slot
  uint64_t cur = 0u, end = range;  // key range still to sort, relative to lo; counted up to end
  uint32_t done = 0u;
  auto load = [&](uint32_t i0, uint32_t (&key)[U], uint32_t* val) {
    uint32_t src[U];
#pragma unroll
    for (int u = 0; u < U; ++u) src[u] = 0u;
    for (uint32_t st = top; st > 0u; st >>= 1) {
#pragma unroll
      for (int u = 0; u < U; ++u) src[u] += lds.poff[src[u] + st] <= i0 + u * THREADS + tid ? st : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = i0 + u * THREADS + tid, at = lds.psrc[src[u]] + i;
      key[u] = i < len ? keys[at] - lo : 0xFFFFFFFFu;
      if (KV && val) val[u] = i < len ? vals[at] : 0u;
    }
  };
  while (done < len) {
    int sh = 0;
    while (((end - cur - 1u) >> sh) > 255u) ++sh;
    __syncthreads();
    for (uint32_t i = tid; i < 256u; i += THREADS) h[i] = 0u;
    __syncthreads();
    for (uint32_t i0 = 0u; i0 < len; i0 += U * THREADS) {
      uint32_t key[U];
      load(i0, key, nullptr);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + u * THREADS + tid < len && key[u] >= cur && key[u] < end) atomicAdd(&h[(uint32_t)((key[u] - cur) >> sh)], 1u);
    }
    __syncthreads();
    if (tid == 0u) {
      uint32_t st = 0u, c = 0u;
      while (st < 256u && c + h[st] <= CAP) c += h[st++];
      if (st == 0u && sh == 0) { c = h[0]; st = 1u; }  // one value: copied, not sorted
      h[256] = st;
      h[257] = c;
    }
    __syncthreads();
    const uint32_t steps = h[256], cnt = h[257];
    if (steps == 0u) {  // the first step alone is too long
      end = cur + (1ull << sh);
      continue;
    }
    const uint64_t stop = cur + ((uint64_t)steps << sh);
    const bool copy = cnt > CAP;
    // the keys in [cur, stop), in the cell's order: into the stage, or one value straight out
    uint32_t at = 0u;
    for (uint32_t i0 = 0u; i0 < len; i0 += U * THREADS) {
      uint32_t key[U], val[U];
      load(i0, key, val);
      uint64_t m[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        m[u] = __builtin_amdgcn_ballot_w64(i0 + u * THREADS + tid < len && key[u] >= cur && key[u] < stop);
      __syncthreads();
      if (lane == 0u) {
#pragma unroll
        for (int u = 0; u < U; ++u) part[u * WAVES + wid] = (uint32_t)__popcll(m[u]);
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        uint32_t p = at + lanes_below(m[u]);
        for (uint32_t w = 0; w < (uint32_t)WAVES; ++w) {
          const uint32_t c = part[u * WAVES + w];
          p += w < wid ? c : 0u;
          at += c;
        }
        if (!((m[u] >> lane) & 1u)) continue;
        if (copy) {
          out[done + p] = key[u] + lo;
          if constexpr (KV) vout[done + p] = val[u];
        } else {
          lds.sort.stage[p] = key[u];
          if constexpr (KV) lds.sort.vstage[p] = val[u];
        }
      }
    }
    __syncthreads();
    if (!copy) {
      const uint32_t lb0 = wid * (64u * IPT) + lane;
      uint32_t k[IPT], v[KV ? IPT : 1];
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        k[j] = lb0 + j * 64u < cnt ? lds.sort.stage[lb0 + j * 64u] : 0xFFFFFFFFu;
        if constexpr (KV) v[j] = lb0 + j * 64u < cnt ? lds.sort.vstage[lb0 + j * 64u] : 0u;
      }
      block_sort_impl<WAVES, IPT, RANK, KV>(lds.sort, k, v, varying_bits<WAVES, IPT>(k, 0u, cnt, lds.sort.scan));
#pragma unroll
      for (int j = 0; j < IPT; ++j)
        if (lb0 + j * 64u < cnt) {
          out[done + lb0 + j * 64u] = k[j] + lo;
          if constexpr (KV) vout[done + lb0 + j * 64u] = v[j];
        }
    }
    done += cnt;
    cur = stop;
    end = range;
  }
}

// Runs of at least this many equal splitters: the value holds at least a sixteenth of the array, and its cell is written by all workgroups together instead of by one.
constexpr uint32_t kCellShareRun = 32;
constexpr uint32_t kMaxCells = 512;

template <int WAVES, int IPT, int RANK, bool KV>
__global__ __launch_bounds__(WAVES * 64, 4) void k_cells(SplitArray a, uint32_t* __restrict__ out, uint32_t* __restrict__ vout,
                                                     const uint32_t* __restrict__ spl, uint32_t P,
                                                     uint32_t* __restrict__ cell_splitters) {
  constexpr uint32_t THREADS = WAVES * 64, CAP = THREADS * IPT;
  __shared__ __align__(16) uint32_t s_stage[CAP];
  __shared__ __align__(16) uint32_t s_vstage[KV ? CAP : 4];
  __shared__ __align__(16) uint32_t s_cnt[WAVES * kBlockRadix];
  __shared__ uint32_t s_poff[THREADS], s_psrc[THREADS], s_scan[WAVES], s_scan2[WAVES];
  __shared__ uint32_t s_nshare, s_share[kMaxCells / kCellShareRun];
  const uint32_t tid = threadIdx.x, b = blockIdx.x, nspl = a.ncells - 1u;
  const CellsLds lds{{s_stage, s_cnt, nullptr, s_scan, s_vstage}, s_poff, s_psrc, s_scan2};
  const uint32_t top = a.ntiles > 1u ? 1u << (31 - __clz((int)(a.ntiles - 1u))) : 0u;
  // the cells written by all workgroups: cell j + 1 for the first j of a long run of equal splitters
  if (tid == 0u) s_nshare = 0u;
  __syncthreads();
  for (uint32_t j = tid; j + kCellShareRun <= nspl; j += THREADS) {
    const uint32_t x = spl[j];
    if (spl[j + kCellShareRun - 1u] == x && (j == 0u || spl[j - 1u] != x)) s_share[atomicAdd(&s_nshare, 1u)] = j;
  }
  const uint32_t lo = b ? spl[b - 1u] : 0u;
  const bool equal = b >= 1u && b < nspl && spl[b] == lo;  // every key of the cell is lo
  const bool shared = equal && b + kCellShareRun - 2u < nspl && spl[b + kCellShareRun - 2u] == lo;
  const uint2 place = cell_pieces<WAVES>(lds, a, b);
  const uint32_t len = place.x, base = place.y;
  uint32_t diff = 0u;
  const bool oversize = len > CAP && !equal;
  if (len && !shared) {
    const gptr<uint32_t> o = gmem(out) + base, vo = gmem(vout) + (KV ? base : 0u);
    if (equal) cell_fill<THREADS, KV>(lds, a, o, vo, top, 0u, len, lo);
    else if (len <= CAP) diff = cell_sort_tile<WAVES, IPT, RANK, KV>(lds, a, o, vo, top, len, lo);
    else
      cell_sort_oversize<WAVES, IPT, RANK, KV>(lds, a, out + base, KV ? vout + base : nullptr, top, len, lo,
                                               (b < nspl ? (uint64_t)spl[b] + 1u : 1ull << 32) - lo);
  }
  // splitters of the output contract whose positions lie in this cell, from LDS (of an oversize cell
  // from memory); the last cell writes those of the empty cells past the end
  if (cell_splitters) {
    const uint32_t q = a.n / P, r = a.n % P;
    if (oversize) __syncthreads();
    for (uint32_t p = max(1u, first_cell_from(base, q, r)) + tid; p < P; p += THREADS) {
      const uint64_t at = (uint64_t)p * q + min(p, r);
      if (at >= a.n) break;
      if (at >= base + len) break;
      const uint32_t i = (uint32_t)at - base;
      cell_splitters[p - 1u] = oversize ? gmem(out)[at] : lo + (diff ? s_stage[i] : 0u);
    }
    if (b == nspl)
      for (uint32_t p = max(1u, first_cell_from(a.n, q, r)) + tid; p < P; p += THREADS) cell_splitters[p - 1u] = 0xFFFFFFFFu;
  }
  const uint32_t nshare = s_nshare;  // written before cell_pieces' barriers
  for (uint32_t i = 0; i < nshare; ++i) {
    const uint32_t j = s_share[i];
    const uint2 c = cell_pieces<WAVES>(lds, a, j + 1u);
    const uint32_t part = (c.x + nspl) / a.ncells;
    cell_fill<THREADS, KV>(lds, a, gmem(out) + c.y, gmem(vout) + (KV ? c.y : 0u), top, min(c.x, b * part),
                           min(c.x, (b + 1u) * part), spl[j]);
  }
}

}  // namespace aps
