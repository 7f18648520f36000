// How many K/V heads a workgroup of the tiled append kernel takes (kv_append.hip).  Plain integer arithmetic, for the launch and for
// a host program alike.
#pragma once

#include <stdint.h>

namespace eco {

constexpr int kAppendThreads = 256;
constexpr int64_t kAppendAtOnceBytes = 256;  // largest row of a head whose block's K (and V) is one 16-byte unit per thread

struct AppendHeads {
  int heads;     // 1, 2 or 4, a divisor of the number of K/V heads
  bool at_once;  // (one head) all loads asked for before the first use
};

// K/V heads per workgroup.  A small call is a chain of round trips, and the less each workgroup brings in the sooner it
// ends: one head, all loads asked for at once, while no more than eight workgroups per CU come of it.  Beyond that the cost
// of finding the block counts, and adjacent heads share it: two, and four from about forty heads' blocks per CU.
// (us, four heads / two / one / one at once, 8 K/V heads of bf16, 128, unless named: 93 tokens 4.95 / 3.66 / 3.10 / 2.92, 512
// 4.59 / 3.94 / 3.77 / 3.44, 2048 6.34 / 5.65 / 5.38 / 5.31, 64 x 20 6.15 / 5.35 / 5.17 / 4.93, 52 heads 5 x 51 6.53 / 5.63 / 5.18 / 5.12;
// 16 x 200 9.11 / 8.69 / 8.62 / 8.74, 4096 10.72 / 9.67 / 9.41 / 9.77, 8192 16.81 / 15.53 / 16.06 / 16.70, 15 x 1024 26.74 / 25.81 /
// 26.86 / 27.27, 256 x 20 19.26 / 17.42 / 18.87 / 18.35, 52 heads 4 x 500 25.99 / 25.10 / 25.90 / 26.28; 4 x 8192 52.79 / 53.65 / 54.10 /
// 56.08.)
// Rows of less than 256 bytes weigh less beside the finding: four heads come earlier, in proportion (8 K/V heads of bf16, two / four, 256
// x 20 tokens: head size 64 7.97 / 7.46, 80 9.21 / 8.81; 64 x 200 10.05 / 9.97 and 12.24 / 12.69).  Rows of 1 KiB are work enough alone: one head, and
// never two; four from 18 blocks of heads per CU, where the rows that they read together count for more (fp32, 256, 4 K/V heads, one /
// two / four: 16 x 512 22.1 / 22.3 / 22.9, 16 x 1000 46.4 / 46.5 / 47.4, 5 x 4096 69.4 / 71.1 / 67.6, 256 x 93 95.0 / 96.8 / 90.4).
inline AppendHeads append_heads(int64_t T, int64_t B, int64_t Hkv, int64_t row_bytes, int64_t num_cu) {
  const int64_t one_head_wgs = (T / 16 + 2 * B) * Hkv, eight_per_cu = 8 * num_cu;
  const bool large_rows = row_bytes >= 1024;
  const bool many = large_rows ? (T / 16 + B) * Hkv > 18 * num_cu : one_head_wgs > 40 * num_cu * (row_bytes < 256 ? row_bytes : 256) / 256;
  if (many && Hkv % 4 == 0) return {4, false};
  if (!large_rows && one_head_wgs > eight_per_cu && Hkv % 2 == 0) return {2, false};
  return {1, one_head_wgs <= eight_per_cu && row_bytes <= kAppendAtOnceBytes};
}

}  // namespace eco
