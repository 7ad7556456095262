// Host side of the two-launch sort (apsort_cells.h): which arrays take it, its tables and launches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "apsort.h"
#include "apsort_cells.h"
#include "apsort_internal.h"

namespace aps {

// Shapes of the split, by array size: waves, keys per lane, sample keys per lane, cells.  Larger
// arrays take larger tiles (a table row per tile, and one round of workgroups on the device), more
// cells (a cell has to fit one tile of k_cells with room for the sample's scatter: 10240 keys, 8192
// pairs, against 400-2300 expected) and a larger sample (8 keys per cell from 400K keys on: the longest cell sets
// the time of the second launch, and at 4 per cell it was half again as long).  Measured, both
// launches, uniform keys:
//     20K   4 keys per lane / 128 cells 14.8 us, 256 cells 15.9
//    100K   4 / 128 19.9, 4 / 256 17.8, 8 / 256 18.3
//    300K   4 / 256 25.3, 8 / 512 21.5
//      1M   8 / 512 35.8, 16 / 512 34.1 (16 waves of 8 keys: 35.5)
// and the two shapes at each bound, mean over ten arrays, uniform / Gaussian keys (pairs alike):
//    48K   4 / 128 16.3 / 16.6, 4 / 256 16.1 / 16.6
//    200K   4 / 256 19.9 / 21.1, 8 / 512 20.3 / 22.2; at 260K 22.0 / 22.4 and 21.2 / 23.6
//    400K   8 / 512 with 4 sample keys per cell 23.4 / 25.3, 16 / 512 25.2 / 28.1; at 500K 24.8 / 28.2
//           and 26.4 / 29.7: by time the line could lie higher, but the cells are then longer for as few
//           sample keys, and nearer to k_cells' tile
struct CellShape {
  size_t max_n;
  uint32_t tile, cells, sample;
};
constexpr CellShape kCellShapes[] = {
    {(size_t)3 << 14, 2048, 128, 1024},
    {(size_t)200000, 2048, 256, 2048},
    {(size_t)400000, 4096, 512, 2048},
    {(size_t)9 << 17, 8192, 512, 4096},
};
// Above these the digit passes take over.  The longest cells come near their tile there (8 sample keys per
// cell and 4 times the mean length of room: one cell in 10^7 longer), and the digit passes skip what
// few-valued keys have in common.  Digit passes / two launches, us: 9 * 2^17 + 1 keys uniform 59.6 / 37.8,
// constant 22.2 / 22.7, bytes 30.0 / 29.8; 5 * 2^18 keys 60.7 / 42.1, 22.0 / 23.1, 30.4 / 30.2.
// Pairs stop earlier: 10 * 2^16 + 1 uniform 57.4 / 36.4, constant 22.0 / 21.3, bytes 29.0 / 26.8, log-uniform
// 51.6 / 52.2; 800K 60.5 / 37.4, 22.0 / 22.5, 29.5 / 29.5, 53.7 / 59.2.
constexpr size_t kCellsMax = (size_t)9 << 17, kCellsMaxPairs = (size_t)10 << 16;
constexpr int kCellIpt = 20, kCellIptPairs = 16;
constexpr uint32_t kPairsSmallMax = 8192;

// Pairs take tiles of at most 4096: twice the work per tile, so half the tile.
static CellShape cell_shape(size_t n, bool pairs) {
  const CellShape* c = kCellShapes;
  while (c < kCellShapes + 3 && n > c->max_n) ++c;
  CellShape r = *c;
  if (pairs) r.tile = std::min(r.tile, 4096u);
  return r;
}

bool cells_sort_size(size_t n, bool pairs) {
  return n > (pairs ? kPairsSmallMax : kSmallSortMax) && n <= (pairs ? kCellsMaxPairs : kCellsMax);
}
bool small_sort_size(size_t n, bool pairs) { return n <= (pairs ? kPairsSmallMax : kSmallSortMax); }

static size_t up256c(size_t x) { return (x + 255) / 256 * 256; }

size_t cells_table_bytes(size_t n, bool pairs) {
  const CellShape c = cell_shape(n, pairs);
  return up256c(sizeof(uint32_t) * c.cells) + up256c(sizeof(uint16_t) * c.cells * ((n + c.tile - 1) / c.tile));
}

// Salt of the sample's positions: the input's address, mixed (the finalizer of SplitMix64).
static uint32_t sample_salt(const void* in) {
  uint64_t x = (uint64_t)(uintptr_t)in;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return (uint32_t)(x >> 32);
}

template <int IPT, int SI, int B, bool KV>
static void launch_split(hipStream_t s, const uint32_t* in, const uint32_t* vin, uint32_t* tmp, uint32_t* vtmp, uint32_t n,
                         uint16_t* table, uint32_t* spl) {
  constexpr uint32_t T = 512 * IPT;
  const dim3 grid((n + T - 1) / T);
  const uint32_t salt = sample_salt(in);
  if (lane_order_ok())
    hipLaunchKernelGGL((k_split<8, IPT, SI, B, SEG_RANK_ATOMIC, KV>), grid, dim3(512), 0, s, in, vin, tmp, vtmp, n, salt,
                       table, spl);
  else
    hipLaunchKernelGGL((k_split<8, IPT, SI, B, SEG_RANK_BALLOT, KV>), grid, dim3(512), 0, s, in, vin, tmp, vtmp, n, salt,
                       table, spl);
}

template <bool KV>
static ap_status enqueue_cells_kv(const uint32_t* in, uint32_t* out, const uint32_t* vin, uint32_t* vout, size_t n, int P,
                                  uint32_t* d_spl, void* tables, uint32_t* tmp, uint32_t* vtmp, hipStream_t s) {
  const CellShape c = cell_shape(n, KV);
  const uint32_t nn = (uint32_t)n, ntiles = (nn + c.tile - 1) / c.tile;
  uint32_t* spl = static_cast<uint32_t*>(tables);
  uint16_t* table = reinterpret_cast<uint16_t*>(static_cast<char*>(tables) + up256c(sizeof(uint32_t) * c.cells));
  prof_begin(AP_KIND_PASS, s);
  if (c.cells == 128) launch_split<4, 2, 128, KV>(s, in, vin, tmp, vtmp, nn, table, spl);
  else if (c.cells == 256) launch_split<4, 4, 256, KV>(s, in, vin, tmp, vtmp, nn, table, spl);
  else if (c.sample == 2048) launch_split<8, 4, 512, KV>(s, in, vin, tmp, vtmp, nn, table, spl);
  else launch_split<KV ? 8 : 16, 8, 512, KV>(s, in, vin, tmp, vtmp, nn, table, spl);
  prof_end(s);
  ap_status st = check_launch(s, "k_split");
  if (st != AP_OK) return st;
  const SplitArray a{tmp, vtmp, table, nn, ntiles, c.tile, c.cells};
  uint32_t* user = P > 1 ? d_spl : nullptr;
  prof_begin(AP_KIND_PASS + 1, s);
  if (lane_order_ok())
    hipLaunchKernelGGL((k_cells<8, KV ? kCellIptPairs : kCellIpt, SEG_RANK_ATOMIC, KV>), dim3(c.cells), dim3(512), 0, s, a, out, vout, spl, (uint32_t)P,
                       user);
  else
    hipLaunchKernelGGL((k_cells<8, KV ? kCellIptPairs : kCellIpt, SEG_RANK_BALLOT, KV>), dim3(c.cells), dim3(512), 0, s, a, out, vout, spl, (uint32_t)P,
                       user);
  prof_end(s);
  return check_launch(s, "k_cells");
}

ap_status enqueue_cells(const uint32_t* in, uint32_t* out, const uint32_t* vin, uint32_t* vout, size_t n, int P,
                        uint32_t* d_spl, void* tables, uint32_t* tmp, uint32_t* vtmp, hipStream_t s) {
  if (vout) return enqueue_cells_kv<true>(in, out, vin, vout, n, P, d_spl, tables, tmp, vtmp, s);
  return enqueue_cells_kv<false>(in, out, nullptr, nullptr, n, P, d_spl, tables, tmp, nullptr, s);
}

template <int WAVES, int IPT>
static void launch_pairs_small(hipStream_t s, const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout,
                               uint32_t n, uint32_t P, uint32_t* spl) {
  if (lane_order_ok())
    hipLaunchKernelGGL((k_sort_pairs_small<WAVES, IPT, SEG_RANK_ATOMIC>), dim3(1), dim3(WAVES * 64), 0, s, kin, vin, kout,
                       vout, n, P, spl);
  else
    hipLaunchKernelGGL((k_sort_pairs_small<WAVES, IPT, SEG_RANK_BALLOT>), dim3(1), dim3(WAVES * 64), 0, s, kin, vin, kout,
                       vout, n, P, spl);
}

// Pairs of at most kPairsSmallMax: one launch (shapes as for keys, enqueue_small_sort).
ap_status enqueue_pairs_small(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout, size_t n, int P,
                              uint32_t* d_spl, hipStream_t s) {
  uint32_t* spl = P > 1 ? d_spl : nullptr;
  prof_begin(AP_KIND_SEG, s);
  if (n <= 2048) launch_pairs_small<4, 8>(s, kin, vin, kout, vout, (uint32_t)n, (uint32_t)P, spl);
  else launch_pairs_small<8, 16>(s, kin, vin, kout, vout, (uint32_t)n, (uint32_t)P, spl);
  prof_end(s);
  return check_launch(s, "k_sort_pairs_small");
}

}  // namespace aps
