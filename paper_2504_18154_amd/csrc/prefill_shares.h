// How a prefill batch of few query tiles is cut into shares of its key steps, one per workgroup (attn_prefill_mfma.hip).
// The items (tile, K/V head) are numbered head after head, tile after tile; an item is worth its key steps and kItemCost
// units in front of them for what it costs besides, and the units of all items are cut into equal shares.  Plain integer
// arithmetic, for the plan kernel and for a host program alike.
#pragma once

#include <math.h>

#if defined(__HIPCC__)
#define ECO_HD __host__ __device__ __forceinline__
#else
#define ECO_HD inline
#endif

namespace eco {

constexpr int kItemCost = 3;
constexpr int kShareMinUnits = 8;   // fewest units of a share
constexpr int kShareMaxRounds = 4;  // most items per workgroup of a batch

// Quotient and root as the rule below needs them: to a few units in the last place, with the bare instructions on the device.
ECO_HD float over(float a, float b) {
#if defined(__HIP_DEVICE_COMPILE__)
  return a * __builtin_amdgcn_rcpf(b);
#else
  return a / b;
#endif
}
ECO_HD float root(float a) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_sqrtf(a);
#else
  return sqrtf(a);
#endif
}

// Workgroups that take shares, 0: the items go through the queues instead, whole.  `units` of all items together, `heaviest`
// and `lightest` item in key steps, n_wgs workgroups, two per CU; n_seqs sequences, of n_tiles query tiles (per K/V head) together.
//
// Shares cost a state of 64 KiB or two per cut, written, read and added up, and even out nothing while they run; items
// cost what the last of them leave idle.  Both are estimated in microseconds: a step takes about 1.06 with a workgroup alone
// on its CU, 1.95 with two; an item that shares its CU with another for s steps ends 0.65 s later; 9 are the start, a first merge
// and some of the 2 to 3 by which the plan takes longer, 0.9 each further piece of the longest item; and a step that no other
// tile of its sequence reads too takes the memory 0.006, whoever computes it, beside what shares write and read in addition.
// Of 222 random batches none takes longer by more than 3% than with whole items where the layers share a plan, 3 do (by 4%)
// where each makes its own; without the last term 40/40 8 x 56+2506 took 99 instead of 87, and 52/52 4 x 100+3000 82 instead of 79.
// Kernel us, items whole / shares (query / K/V heads, new + cached tokens):
//   shares:  64/8 366+4351, 366+11326: 228 / 200    64/8 512+16000: 280 / 264     40/8 32+2000: 36 / 19    40/8 32+16000: 244 / 40
//            40/8 3 x 300+5000: 137 / 111   8/1 5 x 293+8333: 134 / 69    8/1 8192+0: 170 / 148    8/1 2000+0: 36 / 27
//            52/52 200+4000: 72 / 45        8/1 16 x 100+3000: 57 / 41    40/8 584 items of 170 steps, 72 of them in a second
//            round: 427 / 370               64/8 8+30000: 445 / 48
//   whole:   64/8 512+0: 15 / 18            64/8 512+2000: 53 / 53        32/8 4 x 749+89: 40 / 41      40/8 4 x 1024+0: 61 / 63
//            64/8 4 x 256+2000: 79 / 84     64/8 8 x 256+8000: 513 / 525  8/1 16 x 500+500: 35 / 40     64/8 2048+0: 86 / 84
//            40/40 8 x 56+2506: 81 / 91
ECO_HD int share_wgs(int n_items, int units, int heaviest, int lightest, int n_wgs, int n_seqs, int n_tiles) {
  if (heaviest < kShareMinUnits || n_items <= 0 || n_wgs <= 0 || n_tiles <= 0) return 0;
  const float w = (float)n_wgs, u = (float)units, read = 0.006f * u * (n_seqs < n_tiles ? over((float)n_seqs, (float)n_tiles) : 1.f);
  const float work = 1.95f * over(u, w), all = work > read ? work : read;
  // a share is no shorter than what its merge takes: a tile of s steps then has about 0.7 sqrt(s) pieces at most
  const int least = (int)ceilf(root((float)(2 * heaviest))), most = units / (least > kShareMinUnits ? least : kShareMinUnits);
  const int n = most < 1 ? 1 : most < n_wgs ? most : n_wgs;
  const float share = over(u, (float)n);
  const float alone = 1.06f * share, t_share = (alone > all ? alone : all) + 9.f + 0.9f * over((float)heaviest, share);
  float t_items;
  if (n_items <= n_wgs) {
    // the heaviest item, beside the one of rank n_wgs / 2, which is the mean if all are alike, or about this much if not
    const float items = (float)n_items, h = (float)(heaviest + kItemCost), half = 0.5f * w;
    const float rest = items - half;
    float second = 0.f;
    if (rest > 0.f) {
      second = 2.f * over(u, items) * over(rest, items);
      const float low = over(u - half * h, rest);
      second = low > second ? low : second;
      second = second < h ? second : h;
    }
    t_items = 1.06f * h + 0.65f * second;
    t_items = t_items > all ? t_items : all;
  } else {
    // the last round is not full, and it is made of the lightest items
    const int last = n_items % n_wgs;
    t_items = all + (last > 0 ? 0.6f * (1.f - over((float)last, w)) * (float)lightest : 0.f);
  }
  return t_share < 0.97f * t_items ? n : 0;
}

// Whether a batch's key steps may be shared out at all, as far as the host can see: at most n_items items of at most `steps` key
// steps (the width of the block table).  Not for tables so short or batches of so many items that they never would be (more than
// kShareMaxRounds items per workgroup even themselves out), nor for more units than the plan's 32-bit sums hold.
ECO_HD bool may_share_steps(long long n_items, long long steps, int n_wgs) {
  return steps >= kShareMinUnits && n_items <= (long long)kShareMaxRounds * n_wgs && n_items * (steps + kItemCost) <= 0x7fffffff;
}

// Where a share begins: key step `step` of item `item`.
struct Cut {
  int item, step;
};

// The boundary `off` units into an item of `steps` steps.  It leaves two steps on either side, and lies no later than step
// `last` (the one that holds the first row's last key: every row then sees a key in the first step of every piece).
ECO_HD Cut share_cut(int item, int off, int steps, int last) {
  const int j = off - kItemCost;
  if (j < 2) return {item, 0};
  if (j > steps - 2 || j > last) return {item + 1, 0};
  return {item, j};
}

// Boundary r of n, in units of all items together.
ECO_HD int share_begin(int units, int n, int r) { return units / n * r + units % n * r / n; }

// cuts[0..n]: the boundaries, the first at (0, 0), the last behind the last item.  The share that begins the item in which
// share r begins: the last one that begins at the item's step 0 or before it.
ECO_HD int share_that_begins(const Cut* cuts, int r) {
  const int item = cuts[r].item;
  while (cuts[r].item == item && cuts[r].step > 0) --r;
  return r;
}
// The share that ends `item`, of which share r computes a piece: the last one that begins before the next item.
ECO_HD int share_that_ends(const Cut* cuts, int n, int r, int item) {
  while (r + 1 < n && cuts[r + 1].item == item) ++r;
  return r;
}

// Workgroup w of n takes share share_of_wg(w, n): workgroup ids go round-robin to the 8 XCDs, and consecutive shares to one.
ECO_HD int share_of_wg(int w, int n) {
  const int x = w & 7;
  return x * (n >> 3) + (x < (n & 7) ? x : n & 7) + (w >> 3);
}

// The state of an item's piece that share `share` computes: two places per share, since it may hold the end of an item that
// began before it and the beginning of one that goes on behind it.
ECO_HD int piece_slot(int share, int begin) { return 2 * share + (share == begin ? 1 : 0); }

}  // namespace eco
