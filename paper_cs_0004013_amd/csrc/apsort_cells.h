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
// of its stretch, so that a period in the input does not show in the sample.  The salt, made from the
// input's address, keeps the places from being the same for every array of a length: keys that differ
// from all others at known places would put nearly the whole array into one cell.
__device__ __forceinline__ uint32_t sample_pos(uint32_t i, uint32_t stride, uint32_t salt) {
  uint32_t h = i * 0x9E3779B9u + salt;
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
__device__ __forceinline__ void split_sample(const BlockSortLds& lds, gptr<const uint32_t> in, uint32_t n, uint32_t salt,
                                             uint32_t* spl) {
  constexpr int THREADS = WAVES * 64, M = THREADS * SI;
  static_assert(M % B == 0, "whole sample steps per cell");
  static_assert(WAVES > 4, "the tile sort of up to 4 waves needs position words of its own");
  const int tid = threadIdx.x, wid = tid >> 6, lane = tid & 63;
  const uint32_t stride = n / (uint32_t)M;
  uint32_t ks[SI];
#pragma unroll
  for (int j = 0; j < SI; ++j) ks[j] = in[sample_pos((uint32_t)(wid * 64 * SI + j * 64 + lane), stride, salt)];
  const uint32_t first = in[sample_pos(0u, stride, salt)];
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
                                                     uint32_t n, uint32_t salt, uint16_t* __restrict__ table,
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
  split_sample<WAVES, SI, B, RANK>(lds, gin, n, salt, s_spl);
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
  uint32_t* keys;
  uint32_t* vals;
  const uint16_t* table;
  uint32_t n, ntiles, tile, ncells;
};

// The pieces that hold positions i[] of the cell: each is the last one that starts at or before its
// position, found by halvings over the pieces' starts, all positions together so that their reads overlap
// (lanes of neighbouring positions read the same words).  Position i lies at place psrc[piece] + i of the
// split array.
template <int U>
__device__ __forceinline__ void cell_find(const CellsLds& lds, uint32_t top, const uint32_t (&i)[U], uint32_t (&piece)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) piece[u] = 0u;
  for (uint32_t s = top; s > 0u; s >>= 1) {
#pragma unroll
    for (int u = 0; u < U; ++u) piece[u] += lds.poff[piece[u] + s] <= i[u] ? s : 0u;
  }
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
  uint32_t k[I], v[KV ? I : 1], at[I], src[I];
#pragma unroll
  for (int j = 0; j < I; ++j) at[j] = lb0 + j * 64u;
  cell_find<I>(lds, top, at, src);
#pragma unroll
  for (int j = 0; j < I; ++j) src[j] = lds.psrc[src[j]] + at[j];
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
    uint32_t at[4], src[4], val[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) at[u] = i + u * THREADS;
    cell_find<4>(lds, top, at, src);
#pragma unroll
    for (int u = 0; u < 4; ++u) val[u] = at[u] < i1 ? vals[lds.psrc[src[u]] + at[u]] : 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (at[u] < i1) {
        out[at[u]] = key;
        vout[at[u]] = val[u];
      }
  }
}

// A cell longer than one tile whose keys differ: two values that hold more than a tile between them, or keys
// that the sample missed.  Sorted by stable sweeps, one per 8-bit digit that varies (key minus lo, so the
// digits above the cell's range are constant): bucket counts of all digits in one sweep, then every sweep
// ranks tile by tile and writes to the buckets' places.  The sweeps go from the cell's pieces to its part of
// the output and back; an even number of them ends with a copy.  One workgroup does it all, so a long cell
// sets the time of the sort, but every key is read at most six times: a cell of 100K keys takes 0.5 ms, one
// of 9 * 2^17 (keys chosen off the salted positions) 6.6 ms; reading the cell twice for every tile of its
// output, as before, took 455 ms.
template <int WAVES, int IPT, int RANK, bool KV>
__device__ __forceinline__ void cell_sort_oversize(const CellsLds& lds, const SplitArray& a, uint32_t* out_p, uint32_t* vout_p,
                                                   uint32_t top, uint32_t len, uint32_t lo) {
  constexpr int R = kBlockRadix, D = 4, U = 4;
  constexpr int I = 12;  // keys per lane; with all IPT of them the ballot rank spills
  constexpr uint32_t THREADS = WAVES * 64, T = THREADS * I, COPIES = 4, CS = D * R + 1;
  static_assert(2048u + COPIES * CS <= THREADS * IPT, "the tables share the stage");
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
  const gptr<uint32_t> keys = gmem(a.keys), vals = gmem(a.vals), out = gmem(out_p), vout = gmem(vout_p);
  uint32_t* const first = lds.sort.stage;          // [D * R] first position of every bucket
  uint32_t* const running = lds.sort.stage + 1024;  // [R] next free position of every bucket
  uint32_t* const lbase = lds.sort.stage + 1280;    // [R + 1] bucket starts in the tile
  uint32_t* const count = lds.sort.stage + 2048;    // [COPIES * CS]
  uint32_t* const cnt = lds.sort.cnt + wid * R;     // the wave's bucket counts
  __syncthreads();
  for (uint32_t i = tid; i < COPIES * CS; i += THREADS) count[i] = 0u;
  __syncthreads();
  uint32_t* const mine = count + (lane % COPIES) * CS;
  for (uint32_t i0 = 0u; i0 < len; i0 += U * THREADS) {
    uint32_t at[U], src[U], key[U];
#pragma unroll
    for (int u = 0; u < U; ++u) at[u] = i0 + u * THREADS + tid;
    cell_find<U>(lds, top, at, src);
#pragma unroll
    for (int u = 0; u < U; ++u) key[u] = at[u] < len ? keys[lds.psrc[src[u]] + at[u]] - lo : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (at[u] < len) {
#pragma unroll
        for (int d = 0; d < D; ++d) atomicAdd(&mine[d * R + ((key[u] >> (8 * d)) & (R - 1))], 1u);
      }
  }
  __syncthreads();
  uint32_t varies = 0u;  // digits of which no bucket holds every key
  for (uint32_t i = tid; i < D * R; i += THREADS) {
    uint32_t c = 0u;
#pragma unroll
    for (uint32_t q = 0; q < COPIES; ++q) c += count[q * CS + i];
    first[i] = c;
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (!__syncthreads_or(tid < (uint32_t)R && first[d * R + tid] == len)) varies |= 1u << d;
    lds_exclusive_scan<R, (int)THREADS>(first + d * R, lds.sort.scan);
  }
  const uint32_t lb0 = wid * (64u * I) + lane;
  bool in_out = false;  // where the keys are
#pragma unroll 1
  for (uint32_t left = varies; left; left &= left - 1u) {
    const int d = __builtin_ctz(left), shift = 8 * d;
    for (uint32_t b = tid; b < (uint32_t)R; b += THREADS) running[b] = first[d * R + b];
#pragma unroll 1
    for (uint32_t t0 = 0u; t0 < len; t0 += T) {
      uint32_t k[I], v[KV ? I : 1], r[I], at[I], piece[I];
#pragma unroll
      for (int j = 0; j < I; ++j) at[j] = t0 + lb0 + j * 64u;
      if (in_out) {
#pragma unroll
        for (int j = 0; j < I; ++j) k[j] = at[j] < len ? out[at[j]] - lo : 0xFFFFFFFFu;
        if constexpr (KV) {
#pragma unroll
          for (int j = 0; j < I; ++j) v[j] = at[j] < len ? vout[at[j]] : 0u;
        }
      } else {
        cell_find<I>(lds, top, at, piece);
#pragma unroll
        for (int j = 0; j < I; ++j) piece[j] = lds.psrc[piece[j]] + at[j];
#pragma unroll
        for (int j = 0; j < I; ++j) k[j] = at[j] < len ? keys[piece[j]] - lo : 0xFFFFFFFFu;
        if constexpr (KV) {
#pragma unroll
          for (int j = 0; j < I; ++j) v[j] = at[j] < len ? vals[piece[j]] : 0u;
        }
      }
      for (uint32_t b = lane; b < (uint32_t)R; b += 64u) cnt[b] = 0u;
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < I; ++j) {
        const uint32_t b = (k[j] >> shift) & (R - 1);
        if constexpr (RANK == SEG_RANK_ATOMIC) r[j] = rank_slot(cnt, b);
        else r[j] = rank_ballot<kBlockBits>(cnt, b);
      }
      tile_bucket_offsets<R, WAVES>(lds.sort.cnt, lbase, lds.sort.scan);
#pragma unroll
      for (int j = 0; j < I; ++j) {
        const uint32_t b = (k[j] >> shift) & (R - 1);
        r[j] += running[b] + cnt[b] - lbase[b];  // the key's position in the cell
      }
      if (in_out) {
        cell_find<I>(lds, top, r, piece);
#pragma unroll
        for (int j = 0; j < I; ++j) r[j] += lds.psrc[piece[j]];
      }
      const gptr<uint32_t> to = in_out ? keys : out, vto = in_out ? vals : vout;
#pragma unroll
      for (int j = 0; j < I; ++j)
        if (at[j] < len) {
          to[r[j]] = k[j] + lo;
          if constexpr (KV) vto[r[j]] = v[j];
        }
      __syncthreads();  // the buckets' places and counts are read
      for (uint32_t b = tid; b < (uint32_t)R; b += THREADS) running[b] += lbase[b + 1u] - lbase[b];
    }
    in_out = !in_out;
    __syncthreads();  // this sweep's writes before the next one's reads
  }
  if (in_out) return;
  for (uint32_t i0 = 0u; i0 < len; i0 += U * THREADS) {
    uint32_t at[U], src[U];
#pragma unroll
    for (int u = 0; u < U; ++u) at[u] = i0 + u * THREADS + tid;
    cell_find<U>(lds, top, at, src);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (at[u] < len) {
        out[at[u]] = keys[lds.psrc[src[u]] + at[u]];
        if constexpr (KV) vout[at[u]] = vals[lds.psrc[src[u]] + at[u]];
      }
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
    else cell_sort_oversize<WAVES, IPT, RANK, KV>(lds, a, out + base, KV ? vout + base : nullptr, top, len, lo);
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
