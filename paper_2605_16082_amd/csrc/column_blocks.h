// The block table of the layer-parallel column solves (host code only).
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace sdg {

// A block takes 2^log2cols consecutive columns of a cell over the cell's depth, one
// thread per prism.
struct ColTile {
  int32_t base;       // prism slot of the first column's layer 0
  int32_t lbase;      // its level slot
  int32_t col;        // its column slot
  uint16_t depth;     // layers of the cell
  uint16_t log2cols;
};
constexpr int kColSolveMaxLayers = 64;    // deeper meshes take the serial sweeps
constexpr int kColSolveMaxPrisms = 256;   // prisms (threads) of a block
static_assert(kColSolveMaxPrisms / kColSolveMaxLayers >= 4, "16-byte copies need 4 columns a block");

// Column groups of the n_cells cells (of `cell` columns, n_cols columns in all): per
// cell the largest power of two of columns whose prisms fit a block of
// kColSolveMaxPrisms threads (4 columns at 64 layers, where a lane's 16-byte copies still
// hold whole columns; blocks of 512 with twice the columns were 10-15% slower).
// `order` lists the cells deepest first.  max_np: the largest depth << log2cols.
//
// The kernel gives each of the 8 XCDs one contiguous part of the table, so that a
// cell's groups, which share lines, meet in one L2.  Cells of one depth stay in their
// order; otherwise they are dealt to the parts deepest first, back and forth, so that
// every part gets the same share of each depth and takes its deepest cells, the
// longest chains, first.  Against the deepest eighth of all blocks for the first XCD, and so
// on: 68,220 columns of 5 to 60 layers, FP64 4 fields 521 -> 452 us, 1 field 267 -> 216;
// 45,000 columns, all float 2 fields 129 -> 109.
inline std::vector<ColTile> plan_column_blocks(int cell, int n_cols, const std::vector<int32_t>& order,
                                               const std::vector<int32_t>& depth, const std::vector<int32_t>& base,
                                               const std::vector<int32_t>& lbase, int* max_np) {
  *max_np = 0;
  constexpr int kParts = 8;
  const bool uniform = order.empty() || depth[order.front()] == depth[order.back()];
  std::vector<ColTile> part[kParts], table;
  for (size_t i = 0; i < order.size(); ++i) {
    const int32_t k = order[i];
    const int D = depth[k];
    int g = 0;
    while ((2 << g) <= cell && (D << (g + 1)) <= kColSolveMaxPrisms) ++g;
    const int x = (int)(i % kParts);
    std::vector<ColTile>& to = uniform ? table : part[i / kParts % 2 ? kParts - 1 - x : x];
    for (int c0 = 0; c0 < cell && k * cell + c0 < n_cols; c0 += 1 << g)
      to.push_back({base[k] + c0, lbase[k] + c0, k * cell + c0, (uint16_t)D, (uint16_t)g});
    *max_np = std::max(*max_np, D << g);
  }
  if (uniform) return table;
  // the kernel's parts are n / 8 blocks, the first n % 8 of them one more: what a part
  // has beyond that, from its shallow end, goes to the others
  size_t n = 0;
  for (const auto& p : part) n += p.size();
  auto quota = [&](int x) { return n / kParts + ((size_t)x < n % kParts ? 1 : 0); };
  std::vector<ColTile> spare;
  for (int x = 0; x < kParts; ++x)
    for (; part[x].size() > quota(x); part[x].pop_back()) spare.push_back(part[x].back());
  for (int x = 0; x < kParts; ++x)
    for (; part[x].size() < quota(x); spare.pop_back()) part[x].push_back(spare.back());
  table.reserve(n);
  for (const auto& p : part) table.insert(table.end(), p.begin(), p.end());
  return table;
}

}  // namespace sdg
