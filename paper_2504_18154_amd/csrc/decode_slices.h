// How the small-batch decode kernel (attn_any_mfma.hip) cuts a context: which tokens a slice holds, and which entries of
// the sequence's block table a wavefront reads for it - never one behind the sequence's last block, which is the
// caller's to leave unwritten or unbacked.  Plain integer arithmetic, for the kernel and for a host program alike.
#pragma once

#include <math.h>

#if defined(__HIPCC__)
#define ECO_SLICES_HD __host__ __device__ inline
#else
#define ECO_SLICES_HD inline
#endif

namespace eco {

// How long a context's slices are, in blocks, for (bf16, 128) in eight wavefronts (figures in us, 40 query heads on 8 K/V heads).
// A workgroup walks a block in about 0.1; the device streams one (of one K/V head) in 0.0007 and more; slices cost a merge,
// 2.5.  Contexts of up to 1024 tokens stay whole while walking the longest takes no more than that: one of 500 tokens 8.0
// whole, 8.7 in slices of 128; of 777 9.4 and 8.5; 8 x 1000 16.3 and 14.6; 16 x 600 13.9 and 15.2; 16 x 20..1000 14.6 and 12.8.
ECO_SLICES_HD bool whole_context(float longest, float blocks_of_all_heads) {
  const float stream = 0.0007f * blocks_of_all_heads, shortest = 0.1f * 8.f;
  return longest <= 64.f && 0.1f * longest <= (stream > shortest ? stream : shortest) + 2.5f;
}
// The slice that balances a context's walk with its merge (0.13 a slice): sqrt(1.3 blocks), taken a little shorter.  (One context
// in slices of 128 / 256 / 512 tokens, each 1 us faster since: 2000 tokens 11.1 / 11.0 / 12.6, 4000 14.6 / 12.8 / 13.3, 8000
// 18.0 / 17.8 / 16.6.)
ECO_SLICES_HD float least_slice(float blocks) {
#if defined(__HIP_DEVICE_COMPILE__)
  return 1.13f * __builtin_amdgcn_sqrtf(blocks);  // (the bare instruction)
#else
  return 1.13f * sqrtf(blocks);
#endif
}

// Tokens [t0, t1) of slice `sp`; t1 <= t0: there is no such slice.  The last of `max_slices` takes all that is left.
struct Slice {
  int n, t0, t1;  // n: slices of this context
};
constexpr Slice decode_slice(int ctx_len, int split_tokens, int max_slices, int sp) {
  const int want = (ctx_len + split_tokens - 1) / split_tokens, n = want < max_slices ? want : max_slices;
  if (sp >= n) return {n, 0, 0};
  return {n, sp * split_tokens, sp == n - 1 ? ctx_len : (sp + 1) * split_tokens};
}

// The blocks of tokens [t0, t1) (t0 a multiple of 16) go to the wavefronts in turn: entries first + step i, i < n.
struct WaveBlocks {
  int first, step, n;
};
constexpr WaveBlocks wave_blocks(int t0, int t1, int wave, int n_waves) {
  const int blk0 = t0 >> 4, count = ((t1 + 15) >> 4) - blk0;
  return {blk0 + wave, n_waves, wave < count ? (count - wave + n_waves - 1) / n_waves : 0};
}

}  // namespace eco
