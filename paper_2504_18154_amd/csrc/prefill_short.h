// Which (bf16, 128) prefill batches go to the kernel for short contexts (attn_prefill_short.hip), and how they share out its
// wavefronts.  Plain integer arithmetic, for the launch and for a host program alike.
#pragma once

#include <stdint.h>

namespace eco {

enum class PrefillShort {
  kNo,         // the persistent kernel (attn_prefill_mfma.hip)
  kRows64,     // 64 rows per wavefront
  kRows32,     // 32 rows per wavefront
  kSplitKeys,  // the four wavefronts of a workgroup share the keys of 32 rows
};

constexpr int64_t kShortMostKeys = 1024;  // a wavefront's walk: the 64 block ids that a register holds

// `max_ctx`: most tokens of a sequence, cached ones and new ones, as the width of the block table bounds them (the host does not see the
// lengths).  The other side of the line is the persistent kernel with its list of tiles made (ECOSERVE_OPT_PREFILL_REUSE_PLAN): a list of
// its own costs a call 3.5 to 6 us more, but the way, and with it the bits of a result, does not depend on that option.
// Keys are shared while all workgroups run at once, two per CU, and while a walk of a quarter of the keys is no longer than what the persistent kernel takes with
// its key steps shared out (40 on 8, us there / here: 32 + 500 tokens 15.4 / 7.8, 67 + 960 23.8 / 12.3, 32 + 2000 19.2 / 14.4, but 32 + 5300
// 27.6 / 39.8; 8 on 1, 17 x 20 + 2800 22.5 / 24.7; half that where the tiles of a head do not stay with one XCD: 52 on 52, 3 x 66 + 1350 32.3 / 42.2).  Contexts
// of one group of 32 keys have none to share (16 tokens 4.4 against 4.2).  To 1.25 times that many workgroups up to 1536 tokens, and to 1.56 times
// between 256 and 1024 where the tiles of a head stay with one XCD.  Not in the longest contexts, and not beyond 1.25 times, for more than 16 sequences,
// whose K and V come from memory and whose tiles end at many lengths (64 on 8, 17 sequences of 56 to 1652 tokens, eight layers in turn 21.9 / 32.8, one again and again 21.2
// here; 16 on 4, 21 up to 1152 26.8 / 29.0; 8 on 1, 81 of up to 672, 1.5 rounds, 26.7 / 29.0).  Of 8755 random batches of seven head shapes (lengths equal, uniform, lognormal, one in 16 ten times the others), of
// the persistent kernel's time on average, the worst: one round 0.64, 1.22; to 1.25 0.74, 1.22; to 1.56 0.77, 1.10; 20 of 8506 more than 4% slower.  What is left to that
// kernel: 17 sequences and more beyond 1536 tokens (in 1.25 rounds 1024) 0.86, 1.50; the last, 52 on 52, 0.87, 1.18.
//   Rows: no list and no change of tiles, but K and V come once per 32 or 64 rows through the first-level cache, where the
// persistent kernel reads them once per 128 through LDS: the longer the contexts and the fewer the wavefronts, the sooner it wins.
// The line, a context against the cube root of the number of tiles, from 320 random batches (there / here): 52 heads, 128 x 22 tokens 114 / 55,
// 256 x 20 197 / 96, 419 x 36 336 / 204; 40 on 8, 226 x 12 29 / 20, 446 x 80 behind 50..100 334 / 251, 88 x 250 158 / 142; 8 on 1, 28
// x 180 15.0 / 16.5; 16 on 4, 19 x 375 35.9 / 44.0; 40 on 8, 15 385 tokens of 128..4096 504 / 551.  64 rows halve that
// traffic, 32 fill the chip with half the rows (40 on 8, 226 x 12: 20.7 with 32, 22.6 with 64; 446 x 80 308 / 251).
//   Of those 320 batches 228 take the new way: 0.71 of the time on average where the list is made, one 7% slower (8 on 1, 84 x 16 behind up
// to 170: 9.4 / 10.1), the rest no more than 1%; 0.52 where each call makes its own.  Of 4529 of the random ones, 0.62 with 32 rows and 0.73 with 64; of the latter
// 723 eleven are 4 to 21% slower (lengths all equal and a few rows above a multiple of 64: 52 on 52, 39 x 66 behind ~88 53.9 / 65.2).
inline PrefillShort prefill_short(int64_t B, int64_t T, int64_t Hq, int64_t Hkv, int64_t max_ctx, int64_t num_cu) {
  const int64_t tiles = (T * (Hq / Hkv) / 32 + B) * Hkv, wgs = 2 * num_cu;  // tiles of 32 rows, upper bound
  if (tiles >= (int64_t)1 << 30) return PrefillShort::kNo;
  if (max_ctx <= 32) return PrefillShort::kRows32;
  const bool local = Hkv < 8 || Hkv % 8 == 0;  // the tiles of a head stay with one XCD
  const bool few = B <= 16;
  if (tiles <= wgs && 2 * max_ctx <= (!local ? 2 : few ? 4 : 3) * kShortMostKeys) return PrefillShort::kSplitKeys;
  if (max_ctx <= kShortMostKeys && max_ctx * max_ctx * max_ctx <= 6750 * 256 / num_cu * tiles)
    return tiles >= 12 * num_cu && max_ctx > 96 ? PrefillShort::kRows64 : PrefillShort::kRows32;
  if (4 * tiles <= 5 * wgs ? 2 * max_ctx <= (local && few ? 3 : 2) * kShortMostKeys : 16 * tiles <= 25 * wgs && few && local && max_ctx > 256 && max_ctx <= kShortMostKeys)
    return PrefillShort::kSplitKeys;
  return PrefillShort::kNo;
}

}  // namespace eco
