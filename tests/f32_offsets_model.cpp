// Row offsets that the float32 kernels (f32.hip) form, in rows from the first row
// of their buffer, over window lengths, block positions and lanes; prints the
// number that f32_offsets.h does not allow for. At the largest row stride its
// rule lets through, every offset must stay inside what a buffer reaches: rows
// of the sequence below it, others past its end (a negative one as unsigned).
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "f32_offsets.h"

namespace fo = sa::f32_offsets;

static long cases = 0, violations = 0;

static int acc_row(int v, int h) { return (v & 3) + 8 * (v >> 2) + 4 * h; }

static void check(const char* what, int w2, int i0, long long row, int limit) {
  ++cases;
  // the largest row that fits, a multiple of the 16 bytes of a load
  const long long rsb = fo::kReach / limit / 16 * 16;
  const long long off = row * rsb, last = off + rsb;  // any column of the row
  const bool ok = row >= 0 ? last <= fo::kReach && last <= 0x7fffffffLL
                           : off >= -0x80000000LL && (off & 0xffffffffLL) >= fo::kReach;
  if (!ok && ++violations <= 20) std::printf("%s w2=%d i0=%d: row %lld of %d\n", what, w2, i0, row, limit);
}

int main() {
  for (int w2 = 1; w2 <= 300; ++w2) {
    const int lw = fo::row_bits(w2), SP = 32 >> lw, tmask = (1 << lw) - 1;
    const int groups = lw == 5 ? (w2 + 31) / 32 : 1, WT = lw == 5 ? 32 * groups : 1 << lw;
    for (int r = 0; r < 32; ++r) {
      check("row operand", w2, 0, r, fo::kBlockRows);
      check("query of a row", w2, 0, r >> lw, fo::kBlockRows);
      for (int h = 0; h < 2; ++h) check("transposed operand", w2, 0, acc_row(r & 15, h), fo::kBlockRows);
    }
    for (int i0 = 0; i0 < 400; ++i0)
      for (int g = 0; g < groups; ++g) {
        if (w2 <= 128) {  // query side: the lane's k-row, from the first the queries see
          const int k0 = std::max(0, i0 - WT + 1);
          for (int c = 0; c < 32; ++c) {
            const int t0 = (c & tmask) + 32 * g, kk = i0 + (c >> lw) - t0;
            if (t0 < w2 && kk >= 0) check("query side k-row", w2, i0, kk - k0, fo::query_rows(w2));
          }
        }
        if (i0 + SP - 1 < 32 * g) continue;  // key side: such blocks are skipped
        const int k0 = std::max(0, i0 - tmask - 32 * g);
        for (int r = 0; r < 32; ++r) {
          const int t = (r & tmask) + 32 * g;
          if (t < std::min(w2, i0 + (r >> lw) + 1))
            check("key side k-row", w2, i0, i0 + (r >> lw) - t - k0, fo::kBlockRows);
        }
        for (int h = 0; h < 2; ++h)
          for (int v = 0; v < 16; ++v) {
            const int tq = ((8 * (v >> 2)) & tmask) + 32 * g;
            check("key side transposed k-row", w2, i0,
                  i0 - k0 + ((8 * (v >> 2)) >> lw) - tq - (v & 3) - 4 * h, fo::kBlockRows);
          }
      }
  }
  // the rule at its edge, and a stride that int offsets of one row pass
  const bool rule = fo::fits(40, fo::kReach / 40) && !fo::fits(40, fo::kReach / 40 + 1) && !fo::fits(40, 1LL << 40) &&
                    fo::query_rows(16) == 40 && fo::query_rows(128) == 129 && fo::fits(129, 32768LL * 4 * 64) &&
                    !fo::fits(129, 33026LL * 4 * 128);
  std::printf("violations: %ld cases: %ld rule: %s\n", violations, cases, rule ? "ok" : "wrong");
  return 0;
}
