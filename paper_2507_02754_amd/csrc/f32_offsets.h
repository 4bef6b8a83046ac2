// How far the row offsets of the float32 kernels (f32.hip) reach.
//
// Those kernels read rows through buffers that start at the first row of a
// block and take signed 32-bit byte offsets from there. An offset of n rows is
// n times the row stride (heads * head_dim elements), so a stride of many heads
// times the rows of a block can pass 31 bits: such shapes take the plain kernels
// (generic.hip, 64-bit indices) instead.
//
// Plain constexpr functions, so that host code evaluates the rule the library uses.
#pragma once

namespace sa {
namespace f32_offsets {

// Bytes a buffer reaches from its first row; any larger offset (a negative one
// as an unsigned number) is past its end and loads as zeros.
constexpr long long kReach = 0x7ffff000;

// k-rows a wavefront gives each query: 8, 16 or 32 of its 32 rows (log2).
constexpr int row_bits(int w2) { return w2 <= 8 ? 3 : w2 <= 16 ? 4 : 5; }

// Rows, forwards or backwards, that an offset of the forward and of the key side
// reaches: 32 keys or 32 k-rows, the k-rows of up to four queries, and the
// columns of the last row. (The query side's own K and V blocks too.)
constexpr int kBlockRows = 40;
// Of the query side: the k-rows its queries see, from the first one's on.
constexpr int query_rows(int w2) {
  const int lw = row_bits(w2), kspan = lw == 5 ? (w2 + 31) / 32 * 32 : 1 << lw;
  const int rows = kspan + (32 >> lw);
  return rows > kBlockRows ? rows : kBlockRows;
}

constexpr bool fits(int rows, long long row_bytes) { return row_bytes <= kReach / rows; }

}  // namespace f32_offsets
}  // namespace sa
