// How the small-batch decode kernel (attn_any_mfma.hip) cuts a context: which tokens a slice holds, and which entries of
// the sequence's block table a wavefront reads for it - never one behind the sequence's last block, which is the
// caller's to leave unwritten or unbacked.  Plain integer arithmetic, for the kernel and for a host program alike.
#pragma once

namespace eco {

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
