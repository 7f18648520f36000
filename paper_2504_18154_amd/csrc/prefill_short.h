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
// between 256 and 1024 (of the time of the better of the others: 513 to 640 tiles, 513..1024 tokens 0.74 to 0.78, 1025..1536 0.71 to 0.88; 641 to 800, 257..512 0.79 to
// 1.01, 513..1024 0.63 to 0.97; 801 to 960, 257..768 0.85 to 1.19; us there / here: 40 on 8, 616 tokens of 63..507 14.7 / 11.7, 64 on 8, 19 x 11 behind
// 672..1345 28.5 / 20.2, 5 on 1, 9 x 528 behind ~80 21.0 / 16.7; not for more than 16 sequences, whose tiles end at many lengths: 64 on 8, 18 of up to 448 tokens 21.9 / 24.8, 8 on
// 1, 81 of up to 672 26.7 / 29.0).
//   Rows: no list and no change of tiles, but K and V come once per 32 or 64 rows through the first-level cache, where the
// persistent kernel reads them once per 128 through LDS: the longer the contexts and the fewer the wavefronts, the sooner it wins.
// The line, a context against the cube root of the number of tiles, from 320 random batches (there / here): 52 heads, 128 x 22 tokens 114 / 55,
// 256 x 20 197 / 96, 419 x 36 336 / 204; 40 on 8, 226 x 12 29 / 20, 446 x 80 behind 50..100 334 / 251, 88 x 250 158 / 142; 8 on 1, 28
// x 180 15.0 / 16.5; 16 on 4, 19 x 375 35.9 / 44.0; 40 on 8, 15 385 tokens of 128..4096 504 / 551.  64 rows halve that
// traffic, 32 fill the chip with half the rows (40 on 8, 226 x 12: 20.7 with 32, 22.6 with 64; 446 x 80 308 / 251).
//   Of those 320 batches 228 take the new way: 0.71 of the time on average where the list is made, one 7% slower (8 on 1, 84 x 16 behind up
// to 170: 9.4 / 10.1), the rest no more than 1%; 0.52 where each call makes its own.
inline PrefillShort prefill_short(int64_t B, int64_t T, int64_t Hq, int64_t Hkv, int64_t max_ctx, int64_t num_cu) {
  const int64_t tiles = (T * (Hq / Hkv) / 32 + B) * Hkv, wgs = 2 * num_cu;  // tiles of 32 rows, upper bound
  if (tiles >= (int64_t)1 << 30) return PrefillShort::kNo;
  if (max_ctx <= 32) return PrefillShort::kRows32;
  const bool local = Hkv < 8 || Hkv % 8 == 0;  // the tiles of a head stay with one XCD
  if (tiles <= wgs && max_ctx <= (local ? 2 : 1) * kShortMostKeys) return PrefillShort::kSplitKeys;
  if (max_ctx <= kShortMostKeys && max_ctx * max_ctx * max_ctx <= 6750 * 256 / num_cu * tiles)
    return tiles >= 12 * num_cu && max_ctx > 96 ? PrefillShort::kRows64 : PrefillShort::kRows32;
  if (4 * tiles <= 5 * wgs ? 2 * max_ctx <= (local ? 3 : 2) * kShortMostKeys : 16 * tiles <= 25 * wgs && B <= 16 && max_ctx > 256 && max_ctx <= kShortMostKeys)
    return PrefillShort::kSplitKeys;
  return PrefillShort::kNo;
}

}  // namespace eco
