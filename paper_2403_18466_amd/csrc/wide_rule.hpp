// wide_rule.hpp -- launch sizes of the wide network's step and 16-bit adjoint,
// and which of the step's two 16-bit kernels runs (host arithmetic only).
#pragma once

namespace lbm {

// The kernel by row items (wide.hpp): one workgroup of eight wavefronts per
// compute unit (the LDS holds one), every wavefront `per` items of 64 nodes of
// one row.
constexpr int kWideItemWaves = 8;
struct WideItemLaunch {
  long long nb, per;
};
inline WideItemLaunch wide_item_launch(long long nitems, int ncu) {
  long long nb = ncu;
  const long long cap = (nitems + kWideItemWaves - 1) / kWideItemWaves;
  if (nb > cap) nb = cap;
  if (nb >= 16) nb -= nb % 8;
  return {nb, (nitems + nb * kWideItemWaves - 1) / (nb * kWideItemWaves)};
}

inline long long wide_row_items(long long batch, int nx, int ny, int nz) {
  return batch * ((nx + 63) / 64) * ny * nz;
}

// The row kernel's time goes with the items per wavefront, in whole rounds (D3Q19
// 31 us each, D2Q9 28.5); the block kernel's with the blocks of 64 nodes, 9.8 and
// 9.0 us for two per compute unit, in parts of a round too (one workgroup alone
// on a compute unit is faster), and a fifth of that for the start.  So the
// blocks win on small grids, where rows are no multiple of 64, and where the
// items leave part of their last round empty.  us per step, rows / blocks, bf16:
// D3Q19 32^3 29.4 / 12.5, 44^3 60.2 / 31.0, 56^3 64.2 / 53.8, 60^3 62.7 / 68.3,
// 64^3 64.7 / 79.1, 100^3 305 / 294, 112^3 398 / 408, 131 x 150 x 117 624 / 687;
// D2Q9 333^2 55.6 / 32.4, 96 x 2048 57.5 / 55.6, 512^2 59.0 / 73.8, 1024^2 225 /
// 282.  Of 356 sizes, precisions and forcings measured with both kernels the rule
// takes one that is more than 1% slower in nine, and by 4% at most.
inline bool wide_by_blocks(long long batch, int nx, int ny, int nz, int ncu) {
  const long long nblocks = (batch * nx * ny * nz + 63) / 64, round = 2LL * ncu;
  const long long per = wide_item_launch(wide_row_items(batch, nx, ny, nz), ncu).per;
  return 100 * nblocks + 20 * round < 312 * per * round;
}

// The 16-bit adjoint (wide_adj16.hpp).  Its records, 3200 bytes per node, are
// written and read with the non-temporal policy where they exceed the
// last-level cache's 256 MB (less what the fields need).
constexpr long long kWideRecordBytes = 3200;
inline bool wide_adj_streams(long long Np) {
  return Np * kWideRecordBytes > (224LL << 20);
}

// Node ranges of the weight gradients: nsplit of them, four workgroups and one
// slab each, of `per` steps of 32 nodes (the last ones of fewer, or none: the
// number stays a multiple of eight where it exceeds eight, so that a range's
// workgroups share an XCD).  Np: nodes padded to a multiple of 64.
//
// Records in the cache are read back from it, and 32 ranges (half of the chip)
// read as fast as more while their slabs cost less to write and sum: D3Q19
// bf16, whole adjoint, 32 ranges / 64: 32^3 62 / 66 us, 40^3 (205 MB) 99 / 115
// us; with the non-temporal policy 69 and 110 us.  Beyond it 64 ranges, one
// workgroup per compute unit, and non-temporal accesses: 44^3 (273 MB) 135 us
// (149 without, 144 with 32 ranges), 60 x 64 x 52 282 us (361; 301).  At least
// eight steps per range on the small grids.
//
// From 327,680 nodes on 128 ranges, for the length of the float32 sums: against
// float64 sums of short pieces, 128 ranges in a chain of products gave dtheta to
// a relative 2.1-2.4e-7 at 328,000 nodes, 2.5e-7 at 524,000 and 4.7e-7 at 2.1e6;
// 64 of these ranges 1.8-1.9e-7, 2.8-3.3e-7 and 7.2e-7, 128 of them 1.4-1.6e-7,
// 2.0-2.2e-7 and 4.6e-7.
struct WideAdjRanges {
  int per, nsplit;
};
inline WideAdjRanges wide_adj_ranges(long long Np) {
  const long long nsteps = Np / 32;
  const long long most = !wide_adj_streams(Np) ? 32 : (Np <= 327680 ? 64 : 128);
  long long ns = (nsteps + 7) / 8;
  if (ns > most) ns = most;
  if (ns > 8) ns -= ns % 8;
  return {(int)((nsteps + ns - 1) / ns), (int)ns};
}

// Its workspace: the records, then the slabs.
constexpr long long kWideSlabBytes = 546 * 1024;
inline long long wide_adj_workspace_bytes(long long Np) {
  return Np * kWideRecordBytes + wide_adj_ranges(Np).nsplit * kWideSlabBytes;
}

}  // namespace lbm
