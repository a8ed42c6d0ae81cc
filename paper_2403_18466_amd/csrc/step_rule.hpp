// step_rule.hpp -- launch sizes of the learned-collision step with the tanh
// network, and where it takes its small work items (host arithmetic only).
#pragma once

namespace lbm {

// Workgroups for a persistent kernel: as many as there are work units for, a
// multiple of the 8 XCDs when more than 8, and no more than fit on the chip at
// once (occ per compute unit).  Rounded up: rounded down, the last few items
// took a second round (the 2,157 flat items of 600 x 230 nodes, fp32 H = 64: 49 ->
// 29 us).
inline unsigned persistent_grid(int ncu, int occ, long long units_per_block, long long units) {
  if (occ < 1) occ = 1;
  long long want = (long long)ncu * occ;
  if (want > 8) want -= want % 8;
  long long nb = (units + units_per_block - 1) / units_per_block;
  if (nb > 8) nb = (nb + 7) / 8 * 8;
  if (nb > want) nb = want;
  if (nb < 1) nb = 1;
  return (unsigned)nb;
}

// Items of 16 nodes (in workgroups of eight wavefronts) that a wavefront may get,
// in halves, before the 64-node items are the faster form.  With one each the
// 16-node form always is, by 3% and more.  Beyond, four lanes hold each node of a
// 16-node item, so the work at the nodes costs four times as much, and the
// network's share decides; measured on 744 sizes, precisions and forcings, time
// with two items over time with 64-node items: D2Q9 H = 64 0.65-0.94 (three items
// 0.8-1.15), D3Q19 H = 64 fp32 0.83-1.04, unforced 16-bit D3Q19 0.67-0.92 (the
// 64-node form's workgroups of twelve wavefronts leave compute units empty
// there), D2Q9 H = 32 forced 16-bit 0.95-1.01; but D2Q9 H = 32 else 1.08-1.19,
// forced 16-bit D3Q19 0.97-1.22, and D3Q19 H = 32 fp32 0.91-1.0 up to one and a
// half items, 1.06 with two.
constexpr int step_item_halves(int Q, int H, bool fp32, bool forced) {
  if (Q == 9) return H == 64 || (!fp32 && forced) ? 4 : 2;
  if (fp32) return H == 64 ? 4 : 3;
  return forced ? 2 : 4;
}

}  // namespace lbm
