// Prints the column solves' block table of the cells on standard input: a line
// "columns-per-cell columns", then one depth per cell.  Output: "max_np", then one line
// "column depth log2cols" per block.
#include <cstdio>
#include <numeric>

#include "column_blocks.h"

int main() {
  int cell = 0, cols = 0, d = 0;
  if (std::scanf("%d %d", &cell, &cols) != 2) return 1;
  std::vector<int32_t> depth, base, lbase, order;
  for (int32_t b = 0, lb = 0; std::scanf("%d", &d) == 1; b += d * cell, lb += (d + 1) * cell) {
    depth.push_back(d);
    base.push_back(b);
    lbase.push_back(lb);
  }
  order.resize(depth.size());
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return depth[x] > depth[y]; });
  int max_np = 0;
  const auto table = sdg::plan_column_blocks(cell, cols, order, depth, base, lbase, &max_np);
  std::printf("%d\n", max_np);
  for (const auto& t : table) {
    if (t.base != base[t.col / cell] + t.col % cell || t.lbase != lbase[t.col / cell] + t.col % cell) return 2;
    std::printf("%d %d %d\n", t.col, t.depth, t.log2cols);
  }
  return 0;
}
