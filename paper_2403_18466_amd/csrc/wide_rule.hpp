// wide_rule.hpp -- launch sizes of the wide network's step, and which of its
// two 16-bit kernels runs (host arithmetic only).
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

}  // namespace lbm
