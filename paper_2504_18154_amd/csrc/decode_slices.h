// How the small-batch decode kernel (attn_any_mfma.hip) cuts a context: which tokens a slice holds, and which entries of
// the sequence's block table a wavefront reads for it - never one behind the sequence's last block, which is the
// caller's to leave unwritten or unbacked; and which batches it takes.  Plain arithmetic, for the kernel, its launch and for a host
// program alike.
#pragma once

#include <math.h>
#include <stdint.h>

#include <algorithm>

#if defined(__HIPCC__)
#define ECO_SLICES_HD __host__ __device__ inline
#else
#define ECO_SLICES_HD inline
#endif

namespace eco {

// a / b, to a few units in the last place on the device.
ECO_SLICES_HD float quotient(float a, float b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return a * __builtin_amdgcn_rcpf(b);
#else
  return a / b;
#endif
}

// How long a context's slices are, in blocks, for (bf16, 128) in eight wavefronts (figures in us, 40 query heads on 8 K/V heads).
// A workgroup walks a block in about 0.1; the device streams one (of one K/V head) in 0.0007 and more; slices cost a merge,
// 2.5 (when these lines were drawn; it takes 1 to 2 less now, and so do the figures of what is cut).  Contexts of up to 1024 tokens stay whole while walking the longest takes no more than that: one of 500 tokens 8.0
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

// Balanced slices (balanced_slice_blocks in the kernel's file): contexts of nb blocks each, `longest` and `sum` of them, on `slots`
// workgroups of W wavefronts per K/V head.  The slice tried first, in blocks; the slices of a context; the slice tried next, where
// there are more of them than workgroups and the longest context is still cut.
ECO_SLICES_HD int first_balanced_slice(int longest, int sum, int Hkv, int slots, int W) {
  if (W == 8 && whole_context((float)longest, (float)sum * (float)Hkv)) return longest > 1 ? longest : 1;  // (four: two workgroups per CU, see small_decode)
  const float least = least_slice((float)longest) - 0.5f * (float)W, even = quotient((float)sum, (float)slots);
  return ((int)(least > even ? least : even) / W + 1) * W;
}
ECO_SLICES_HD int balanced_slices_of(int nb, int st) {
  // (exact up to 2^21 blocks; a slice too many would find nothing left to do, and the last of one too few takes the rest)
  return (int)quotient((float)nb + ((float)st - 0.5f), (float)st);
}
ECO_SLICES_HD int next_balanced_slice(int st, int W) { return st + ((st >> 2) > W ? st >> 2 : W) / W * W; }

// Tokens [t0, t1) of slice `sp`; t1 <= t0: there is no such slice.  The last of `max_slices` takes all that is left.
struct Slice {
  int n, t0, t1;  // n: slices of this context
};
constexpr Slice decode_slice(int ctx_len, int split_tokens, int max_slices, int sp) {
  const int want = (ctx_len + split_tokens - 1) / split_tokens, n = want < max_slices ? want : max_slices;
  // (without the number of slices, whose division a kernel need not wait for)
  if (sp >= max_slices || (int64_t)sp * split_tokens >= ctx_len) return {n, 0, 0};
  const int t0 = sp * split_tokens;
  return {n, t0, sp == max_slices - 1 || ctx_len - t0 <= split_tokens ? ctx_len : t0 + split_tokens};
}

// The blocks of tokens [t0, t1) (t0 a multiple of 16) go to the wavefronts in turn: entries first + step i, i < n.
struct WaveBlocks {
  int first, step, n;
};
constexpr WaveBlocks wave_blocks(int t0, int t1, int wave, int n_waves) {
  const int blk0 = t0 >> 4, count = ((t1 + 15) >> 4) - blk0;
  return {blk0 + wave, n_waves, wave < count ? (count - wave + n_waves - 1) / n_waves : 0};
}

// ---- how the host has the decode kernel of attn_any_mfma.hip launched ---------------------------

// Wavefronts of a decode workgroup: eight while two blocks of K and V fit beside the rest in 256 registers.
constexpr int decode_wavefronts(int D, int elem_bytes) { return D > (elem_bytes == 4 ? 128 : 192) ? 4 : 8; }

// A slice of up to so many rounds of the wavefronts is a short one; so many tokens are it at most, in eight wavefronts.
constexpr int kShortRounds = 4, kShortSlice = kShortRounds * 8 * 16;

struct SmallDecode {
  int32_t split_tokens, n_split;  // as launch_decode_any takes them
};

// Contexts up to 1024 tokens stay whole (no merge); longer ones are cut into slices of 256 tokens, or of 512 or 1024
// when that already makes enough workgroups.  (8 K/V heads, bf16, 128, us in slices of 256 / 512 / 1024: one sequence of 2000
// tokens 9.6 / 10.3 / 12.7, of 8000 14.9 / 12.6 / 13.8; 4 x 2000 11.1 / 10.9 / 13.3.)
inline int32_t decode_any_split_tokens(int32_t B, int32_t Hkv, int32_t max_ctx_len, int32_t num_cu) {
  int32_t st = max_ctx_len > 1024 ? 256 : 1024;
  while (st < 1024 && (int64_t)B * Hkv * ((max_ctx_len + st - 1) / st) > num_cu / 2) st *= 2;
  return st;
}

// For every other layout: contexts are cut, into slices of whole rounds of the wavefronts, where that makes no more than one
// workgroup per CU and the walk it saves is worth a merge.  A block's walk takes 0.012 us per KiB of it in bf16, 0.018 in fp32 (one of
// 700 tokens against one of 50: 64 0.05 and 0.16, fp32 128 0.28, 192 0.13, 256 0.21 and 0.57 us a block); a merge 2.7
// (1.8 in fp32), more for large heads, and 0.13 a slice (all figures here are from before it became 1 to 2 us cheaper).  Us per call whole / cut: fp32, 64, 2 K/V heads: 1 x 700 tokens 11.2 / 7.6, 16 x 700 11.5 / 9.0; fp32, 128, 3:
// 1 x 400 14.2 / 9.5, 4 x 37..708 15.6 / 10.4, 8 x 3000 33.6 / 22.6; fp32, 256, 2: 16 x 700 41.4 / 21.2; bf16, 192, 2: 16 x 700 16.7 / 12.8; bf16, 256, 1:
// 1 x 200 11.7 / 13.1, 1 x 400 14.3 / 13.6, 64 x 800 27.1 / 21.3; bf16, 96, 2: 16 x 700 8.4 / 9.0; 64, 8: 1 x 700 6.6 whole.
//   Slices beyond 1024 tokens are no longer than the uniform ones would be (bf16, 32, 1 x 2000: 256 tokens 7.1, 512 7.6; 96, 2 x 4000: 256
//   10.3, 384 11.1), and a slice is as much shorter than the context as half a merge's walk (fp32, 128, 16 K/V heads, 8 x 300 tokens:
//   whole 17.2, 256 and the rest 18.5; 96, 32 heads, 4 x 300 14.1 / 15.5).  bf16 heads above 192 merge four states at a time: no
//   less than 256 tokens beyond 1024 (256, 1 x 1100: 256 tokens 15.1, 128 16.4; 1 x 4000 18.6, 192 21.3; but 1 x 700 15.2, 128 14.0).
//   Against the best of nine forced lengths of slices, 1558 batches of 15 layouts: 2.3% longer on average in bf16, 4.1% in fp32 (8.4 and 32
//   with the uniform slices alone, 2.6 and 4.2 without these three rules).
inline SmallDecode any_decode(int32_t B, int32_t Hkv, int32_t D, int32_t elem_bytes, int32_t max_ctx_len, int32_t num_cu) {
  const int32_t W = decode_wavefronts(D, elem_bytes), nb = (max_ctx_len + 15) / 16;
  const int64_t slots = num_cu / ((int64_t)B * Hkv);
  const float large = std::max(1.f, (float)D / 192.f), walk = (elem_bytes == 2 ? 0.012f : 0.018f) * (float)(32 * D * elem_bytes) / 1024.f;
  const float merge = (elem_bytes == 2 ? 2.7f : 1.8f) * large, state = 0.13f * large;
  const int32_t uniform = decode_any_split_tokens(B, Hkv, max_ctx_len, num_cu), n_uniform = (max_ctx_len + uniform - 1) / uniform;
  if (slots > 1 && walk * (float)(nb - W) > merge) {
    const int64_t least = std::max<int64_t>((int64_t)sqrtf(state / walk * (float)nb), (nb + slots - 1) / slots);
    int32_t st = (int32_t)std::min<int64_t>((least + W - 1) / W * W, 64) * 16;
    if (max_ctx_len > 1024 && n_uniform <= slots) st = std::min(st, uniform);
    if (max_ctx_len > 1024 && elem_bytes == 2 && D > 192 && (max_ctx_len + 255) / 256 <= slots) st = std::max(st, 256);
    const int32_t n = (max_ctx_len + st - 1) / st;
    if (max_ctx_len > 1024 || walk * (float)(nb - st / 16) > 0.5f * merge + state * (float)n) return {st, n};
  }
  return {uniform, n_uniform};
}

// For (bf16, 128): wavefronts per (sequence, K/V head) with which decode_short_kernel takes a batch whole, 0 if it does not.  The host knows the longest
// context, not the others, and walking it is the launch's time at least (20 us for 1700 tokens by four wavefronts) however short those are: the line lies
// where no lengths make it cost more than a few percent.  From 18800 random batches of seven head shapes, up to 9000 tokens: lengths equal, uniform from 1/2, 1/8 and 1/64 of the
// longest on, lognormal around 1/3, 1/6 and 1/10 of it, and one sequence in 16 ten times as long as the others.  Of the time of the other kernels, with
// the append fused in (mean, the worst; of 7700 without the append 0.79, 1.11, of 3600 against the persistent kernel's measured shares 0.70, 1.05):
//   Few (sequence, K/V head)s, up to where contexts cut into slices, or eight wavefronts to a context, end sooner: 0.80, 0.97.
//   129 to 256, up to 384 tokens: 0.89, 1.00.  Beyond, slices even out ragged lengths: 385 to 512 0.99, 1.11; 513 to 1024 1.02, 1.33; 1025 to 4096 1.02, 2.15
// (0.87 where all are as long, 1.22 where most are a sixth and less of it).
//   257 to 320, up to 640: 0.85, 1.07; 641 to 1024 0.85, 1.14; 1025 to 2048 1.01, 1.58.
//   More: against the persistent kernel, whose launch is even whatever the lengths.  321 to 768, up to 1280: 0.75, 1.03; 1281 to 2048 0.92, 1.20; 2049 to
// 4096 1.04, 1.63.  769 to 2048, up to 1664: 0.70, 1.06; 1665 to 2048 0.92, 1.11; 2049 to 4096 0.98, 1.32.  In the largest batches its start and end no
// longer count.  2049 to 3072, up to 1280: 0.71, 1.04; 1281 to 2048 0.91, 1.07, lengths all equal 1.03.  From 3073 on, up to 832: 0.72, 1.05; 833 to 1280 0.89, 1.07,
// equal 1.03.
//   One wavefront is the cheapest for contexts of two blocks, and for longer ones while enough others run (768 to 1024: 97..128 tokens 1.00, two
// 1.02, 193..256 1.08 / 1.00; 6144 to 8192: x 257..512 1.00 / 1.02); two likewise (385 to 512: 97..192 1.02, four 1.00; 769 to 1024: 385..512 1.00 / 1.14; 2048 to
// 3072: 513..768 1.01 / 1.01).
inline int32_t decode_short(int32_t B, int32_t Hkv, int32_t max_ctx_len, int32_t num_cu) {
  const int64_t pairs = (int64_t)B * Hkv, cu = num_cu, tokens = max_ctx_len;
  const int64_t most = 32 * pairs <= cu ? 512 : 4 * pairs <= cu ? 384 : 2 * pairs <= cu ? 320 : pairs <= cu ? 384 : 4 * pairs <= 5 * cu ? 640
                     : pairs <= 3 * cu ? 1280 : pairs <= 8 * cu ? 1664 : pairs <= 12 * cu ? 1280 : std::min<int64_t>(832, 32000 * cu / pairs);
  if (tokens > most) return 0;
  return tokens <= 32 || tokens * cu <= 32 * pairs ? 1 : tokens <= 96 || tokens * cu <= 96 * pairs ? 2 : 4;
}
// Whether its workgroups are handed out by length, longest first: more of them than CUs, and contexts long enough for the end of the launch to
// show it (in order of the batch / of length, of the best: 385 to 512 (sequence, head)s, up to 192 tokens 1.00 / 1.07, 193..256 1.08 / 1.00; 1024 x 65..128 1.00 / 1.02;
// 4096 x 33..64 1.00 / 1.01, 65..128 1.10 / 1.00).
inline bool decode_short_ordered(int64_t pairs, int32_t max_ctx_len, int32_t num_cu) {
  return pairs > num_cu && max_ctx_len > (pairs > (int64_t)4 * num_cu ? 96 : 192);
}
// Whether what it writes back goes past the caches: 5 KiB per (sequence, head), which the last-level cache (256 MB) holds until the next step for a few layers,
// not for those of a model, and written back from there it costs more.  1024 x ~103 tokens on 8 K/V heads, 2, 4 and 8 layers, kept / past the caches: 99.9 /
// 104.5, 103.3 / 104.7, 115.7 / 104.9 us a layer; 512 x ~103 60.7 / 61.8, 60.8 / 62.3, 62.8 / 62.4.  With three sets of 2 to 8 layers in turn (1387 batches; of the
// best): 2049 to 4096 (sequence, head)s, up to 96 tokens 1.09 / 1.00, 97..192 1.02 / 1.01, 193..384 1.01 / 1.02; 4097 to 8192, 97..192 1.06 / 1.01, 385..768 1.01 /
// 1.01; 16385 to 32768, 97..192 1.19 / 1.01.
constexpr bool decode_short_stream(int64_t pairs, int32_t max_ctx_len) { return pairs > (max_ctx_len <= 192 ? 2048 : 4096); }

// Whole contexts, longest first, the longer ones cut (decode_short_kernel, kSliced): slices of `blocks` blocks, whole ones first, then what is left of each context.  No
// more than `max_full` whole slices per K/V head come of it, whatever the lengths, and twice as many slots for partial states.
constexpr int32_t kSlicedMostSequences = 256;  // four lengths per lane
// (three per CU: as many workgroups as run there at a time, and the rests follow them)
inline int32_t sliced_most_full(int32_t, int32_t Hkv, int32_t num_cu) { return 3 * num_cu / Hkv; }
struct SlicedContexts {
  int blocks;
  float per_block;
  ECO_SLICES_HD int full(int nb) const {  // whole slices of a context of nb blocks, at least one block being left over
    if (nb <= blocks) return 0;
    const int f = (int)(((float)nb - 0.5f) * per_block);
    return (int64_t)f * blocks >= nb ? f - 1 : f;
  }
  ECO_SLICES_HD int size_class(int left) const {  // 0 to 15
    const int c = (int)((float)left * per_block * 15.f);
    return c < 15 ? c : 15;
  }
};
ECO_SLICES_HD SlicedContexts sliced_contexts(int sum, int max_full, int W) {
  constexpr int kLeast = 24;
  const int even = max_full > 0 ? (sum + max_full - 1) / max_full : sum, least = even > kLeast ? even : kLeast;
  const int blocks = (least + W - 1) / W * W;
  return {blocks, quotient(1.f, (float)blocks)};
}

// For (bf16, 128), batches that decode_short leaves: how decode_any_kernel takes a small one, n_split 0 if it does not.  It needs no numbering of the batch and no
// second launch, which is what such a batch spends its time on in the persistent kernel.
//   (The lines of this rule were drawn against the persistent kernel and with a merge that took 1 to 2 us longer; what it leaves now goes to decode_sliced, against which only
//   one context was measured again.)
//   Several sequences, one of them of more than 768 tokens, and eight workgroups (one per CU) or more per five (sequence, K/V
//   head)s: balanced slices.  Us per call before (uniform slices or the persistent kernel) / balanced: 64 query heads on 8, 16 x
//   20..2000 tokens 18.4 / 14.5, 8 x 20..8000 19.2 / 14.6; 8 on 1, 64 x 1000..8000 38.5 / 28.8; 32 on 8, 9 x
//   1196..9574 35.8 / 29.0; 40 on 8, 18 x 116..935 15.6 / 14.3, 8 x 1000 16.0 / 13.9, 16 x 1000 18.9 / 18.4, 16 x 2000 29.2 / 27.8, 20 x 2000 38.9 / 32.8, 20 x
//   100..3000 30.2 / 26.1.  Finding the slices takes half a microsecond, and just above 768 tokens a batch whose longest context
//   is alone gains what an evenly ragged one loses (16 x 50..800 13.7 / 14.2, 15 x 50 and one of 800 12.4 / 10.0; 52 on 52, 1000 and 2000
//   20.1 / 20.5).  Fewer spare workgroups even out too little (24 x 1000..10000 84 / 98), and from 400 MB on the persistent kernel's stream
//   is the faster one (16 x 8000 93 / 99, both without the non-temporal hint; 15 x 1142..9140, forced, 51.8 / 51.7).
//   No balancing where every sequence may have as many slices as one of max_ctx_len tokens gets for itself: the slices of
//   balanced_slice_blocks for that (1 x 777: 9.4 / 8.3, 1 x 1000: 10.6 / 8.6, 1 x 16000: 21.3 / 20.9; 5 on 1, 13 x 745..5960 17.3 / 12.7).
//   Else uniform slices if all workgroups run at once, one of eight wavefronts per CU (us per call persistent / here: 16 x 1000
//   tokens 20.7 / 14.1).
//   Else balanced slices for two workgroups of four wavefronts per CU, all of which run at once too, with as many to spare, up
//   to 300 MB (persistent / here: 40 x 100..1000 27.2 / 24.6, 40 x 20..2000 25.1 / 21.2, 28 x 100..3000 37.5 /
//   33.5, 24 x 100..3000 33.0 / 30.2, 16 query heads on 4, 64 x 100..2000 31.9 / 28.3; 36 x 1500 49.0 / 49.0, 40 x 2000 65.3 / 66.1, 24 x
//   4000 74 / 80; with nothing to spare 64 x 20..2000 33.7 / 39.2; three workgroups and more per CU 40 x 100..1000 28.5).
//   One context too long for the first of these rules comes here too, however long (1 x 40000 52.3 / 43.5, 1 x 75000 75.1 / 64.4; 8 on 1, 1 x 300000 226 / 60,
//   1 x 600000, cut into 171 slices, 252 / 86; 20 on 4, 1 x 150000 91 / 77).  Beyond 600000 tokens of all K/V heads it was the persistent kernel's, then slices of whole blocks
//   handed out by rank (decode_sliced); us persistent / by rank / here: 40 on 8, 1 x 80000 78.6 / 78.5 / 67.2, 1 x 400000 284 / 280 / 269; 64 on 8, 1 x 120000 113 / 104 / 92; 8 on 1, 1 x
//   800000 267 / 219 / 101, 1 x 1500000 320 / 284 / 208; 32 on 32, 1 x 19000 60.0 / 57.1 / 53.4; 52 on 52, 1 x 60000 258 / 253 / 250.  (The non-temporal hint for
//   contexts beyond the last-level cache changed nothing where the slices are uniform.)
inline SmallDecode small_decode(int32_t B, int32_t Hkv, int32_t max_ctx_len, int32_t num_cu) {
  const int64_t pairs = (int64_t)B * Hkv;
  const int32_t nb = (max_ctx_len + 15) / 16, slots = num_cu / Hkv;
  const bool whole = whole_context((float)nb, (float)nb * (float)Hkv);  // (also of more sequences, then)
  if (!whole && slots > 0 && pairs * ((max_ctx_len + 1023) / 1024) <= num_cu) {
    int32_t st = ((int32_t)least_slice((float)nb) + 4) / 8 * 8;  // whole rounds of eight wavefronts
    // no more than 16 slices up to 40 blocks each (the merge adds up eight at a time; 1 x 8000, 64 heads on 8: 21 slices 14.2, 13 12.4, 8 on 1 11.0 / 9.9)
    if (B == 1 && nb <= 16 * 40) st = std::max(st, (nb + 16 * 8 - 1) / (16 * 8) * 8);
    if (B == 1) st = std::max(st, (nb + 8 * slots - 1) / (8 * slots) * 8);
    // slices of 256 tokens for all sooner than balanced ones: no search, and plain loads (40 on 8, 8 x 1000 12.4 balanced, 11.3 so)
    if (B > 1 && st == 8 && B * ((nb + 7) / 8) > slots && B * ((nb + 15) / 16) <= slots) st = 16;
    if (B * ((nb + st - 1) / st) <= slots && (B == 1 || nb > 48)) return {st * 16, (nb + st - 1) / st};
  }
  if (B > 1 && B <= 64 && nb > 48 && 8 * B <= 5 * slots && pairs * max_ctx_len <= 800000) return {0, slots};
  const int32_t st = decode_any_split_tokens(B, Hkv, max_ctx_len, num_cu), n = (max_ctx_len + st - 1) / st;
  if (pairs * n <= num_cu) return {st, n};
  const int32_t slots2 = 2 * num_cu / Hkv;
  if (B <= 64 && 8 * B <= 5 * slots2 && (B == 1 || pairs * max_ctx_len <= 600000)) return {0, slots2};
  return {0, 0};
}

// For (bf16, 128), batches that neither of these takes: whether whole contexts with the longer ones cut have them (else the persistent kernel).  Up to where the
// launch's start and end no longer count beside its stream: at 3120 (sequence, K/V head)s, 52 on 52, 60 x 1500..2000 tokens, the persistent kernel takes 461 us, this one 482.
//   Us per call, fused append, the persistent kernel / here: 40 on 8, 128 x 512..4096 208 / 196, 64 x 20..2000 57.6 / 52.8, 100 x 50..3000 118.8 / 109.3, 256 x 100..1800 190 / 176,
// 127 x 20 and one of 4000 24.0 / 16.2; 64 on 8, 256 x 1024..4096 459.5 / 451.3, 128 x 8192 671 / 672, 8 x 60000 323 / 313; 52 on 52, 24 x 300..3000 185 / 177; 32 on 8, 64 x 4096 183 / 170,
// 84 x 300 and six of 6000 57.9 / 49.7; 8 on 1, 256 x 100..6000 80.4 / 78.0; 5 on 1, 150 x 300..16000 115.2 / 114.8.  That is for caches of a few layers, which the last-level cache holds in
// part: over the 64 layers of a model the first of these batches streams at the same rate by either kernel, and the 256 long contexts are the persistent kernel's with measured shares (below).
//   Whole slices per CU, at most: three, as many workgroups as run there at a time.  Of 60 random batches that come here, of the persistent kernel's time, (two, three, four): up to 1.75
// (sequence, head)s per CU 0.936, 0.934, 0.943 on average, the worst 1.14, 1.05, 1.07; above 0.932, 0.929, 0.936.  (52 on 52, 5 x 5594 143, 131, 130 us, 8 on 1, 256 x 100..6000
// 80.6, 78.0, 80.4, 5 on 1, 150 x 300..16000 118, 115, 116.)  What stays slower than the persistent kernel, by up to 5%, are few long contexts of much the same length, whose rests run one
// to a CU; where one in 16 is long, as the host cannot see, these batches take 10 to 35% less than there.
inline bool decode_sliced(int32_t B, int32_t Hkv, int32_t num_cu) { return B <= kSlicedMostSequences && (int64_t)B * Hkv <= (int64_t)8 * num_cu; }
// A context that asks for shares by each XCD's measured speed keeps the persistent kernel for its longest launches: the shares take 1 to 3% off a stream, which is more
// than the launch of the merge and the uneven end cost once the stream is long.  Us per call with such shares, the persistent kernel / here: 64 on 8, 256 x 1024..4096
// 447 / 449, 200 x 1024..8300 624 / 636, 16 x 30000..60000 482 / 493; 32 on 32, 64 x 500..4096 392 / 398; 40 on 8, 160 x 512..4096 252 / 251, 128 x 512..4096 206 / 199.  (With
// equal shares the first of these take 456, 631, 484, 397, 257: all but the third longer than here.)
inline bool adaptive_stream(int32_t B, int32_t Hkv, int32_t max_ctx_len, int32_t num_cu) { return (int64_t)B * Hkv * max_ctx_len > (int64_t)20000 * num_cu; }

}  // namespace eco
