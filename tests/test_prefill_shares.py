"""csrc/prefill_shares.h, the arithmetic by which a prefill batch of few query tiles is cut into shares of its key steps,
compiled for the host: over random batches every key step of every item is computed once, no piece is empty or begins behind
what its first row sees, and the pieces of a cut item name the same states and the same counter, which no other item uses."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <map>
#include <random>
#include <vector>
#include "prefill_shares.h"
using namespace eco;

static int fail(const char* what) { return std::printf("%s\n", what), 1; }

int main() {
  std::mt19937 rng(1);
  long cut_items = 0;
  for (int it = 0; it < 3000; ++it) {
    const int tiles = 1 + rng() % (it % 3 ? 12 : 200), heads = 1 + rng() % (it % 2 ? 8 : 52), longest = 1 + (rng() % 4 ? rng() % 40 : rng() % 800);
    std::vector<int> steps(tiles), last(tiles), sum(tiles + 1, 0);  // last: the step that holds the first row's last key
    for (int t = 0; t < tiles; ++t) {
      steps[t] = 1 + rng() % longest;
      last[t] = std::max(0, steps[t] - 1 - (int)(rng() % 3));
      sum[t + 1] = sum[t] + steps[t] + kItemCost;
    }
    const int units = sum[tiles] * heads, items = tiles * heads;
    const int n = std::min(1 + (int)(rng() % 512), std::max(units / kShareMinUnits, 1));
    std::vector<Cut> cuts(n + 1);
    for (int r = 0; r <= n; ++r) {
      const int u = share_begin(units, n, r), g = u / sum[tiles], v = u - g * sum[tiles];
      const int t = std::min<int>(std::upper_bound(sum.begin(), sum.end(), v) - sum.begin() - 1, tiles - 1);
      cuts[r] = r == n ? Cut{items, 0} : share_cut(g * tiles + t, v - sum[t], steps[t], last[t]);
    }
    std::vector<int> taken(n, 0);
    for (int w = 0; w < n; ++w) {
      const int r = share_of_wg(w, n);
      if (r < 0 || r >= n || taken[r]++) return fail("a share without, or with two workgroups");
    }
    std::vector<std::vector<int>> seen(items);
    for (int i = 0; i < items; ++i) seen[i].assign(steps[i % tiles], 0);
    std::map<int, int> slot_used, counter_of, item_of_counter;
    std::map<int, std::vector<int>> slots;
    for (int r = 0; r < n; ++r) {
      const int first = cuts[r].item, end = cuts[r + 1].step, final = cuts[r + 1].item - (end == 0 ? 1 : 0);
      const int begin0 = first < items ? share_that_begins(cuts.data(), r) : r;
      for (int i = first; i <= final; ++i) {
        const int a = i == first ? cuts[r].step : 0, b = i == final && end > 0 ? end : steps[i % tiles];
        if (a >= b) return fail("an empty piece");
        if (a > 0 && a > last[i % tiles]) return fail("a piece that begins behind what its first row sees");
        for (int j = a; j < b; ++j) ++seen[i][j];
        const int begin = i == first ? begin0 : r;
        const int pieces = share_that_ends(cuts.data(), n, r, i) - begin + 1;
        if ((pieces == 1) != (a == 0 && b == steps[i % tiles])) return fail("a whole item in pieces, or a piece taken for a whole");
        if (i != first && i != final && pieces > 1) return fail("a cut item in the middle of a share");
        if (pieces == 1) continue;
        if (slot_used[piece_slot(r, begin)]++) return fail("a state written twice");
        slots[i].push_back(piece_slot(r, begin));
        if (counter_of.count(i) && counter_of[i] != begin * 4096 + pieces) return fail("pieces that do not agree");
        counter_of[i] = begin * 4096 + pieces;
      }
    }
    for (const auto& s : slots) {
      const int begin = counter_of[s.first] / 4096, pieces = counter_of[s.first] % 4096;
      if (item_of_counter[begin]++) return fail("a counter of two items");
      if ((int)s.second.size() != pieces) return fail("a piece missing");
      for (int k = 0; k < pieces; ++k)
        if (s.second[k] != piece_slot(begin + k, begin)) return fail("a state out of order");
      ++cut_items;
    }
    for (const auto& item : seen)
      for (int x : item)
        if (x != 1) return fail("a key step not computed once");
  }
  if (cut_items < 10000) return fail("too few cut items");
  // whole items: tiles too short to cut, full rounds of equal items, many light items; shares: one long item, a bad last round
  if (share_wgs(32, 32 * 5, 2, 2, 512, 1, 32) || share_wgs(512, 512 * 53, 50, 50, 512, 1, 512) || share_wgs(1280, 1280 * 20, 32, 1, 512, 16, 1280)) return fail("shares");
  if (!share_wgs(8, 8 * 253, 250, 250, 512, 1, 1) || !share_wgs(584, 584 * 171, 200, 103, 512, 2, 73)) return fail("no shares");
  // every sum that the plan makes of a batch it may share fits 32 bits: at the line, and beyond it not (2047 tiles of one K/V head
  // behind 68 million cached tokens: the sum of their units wraps around)
  for (long long items : {1LL, 7LL, 512LL, 2047LL, 2048LL}) {
    const long long most = 0x7fffffff / items - kItemCost;
    if (!may_share_steps(items, most, 512) || may_share_steps(items, most + 1, 512)) return fail("units that 32 bits do not hold");
  }
  if (may_share_steps(2047, 68000000 / 64 + 1, 512)) return fail("a sum that wraps around");
  if (may_share_steps(2049, 100, 512) || may_share_steps(8, kShareMinUnits - 1, 512) || !may_share_steps(2048, 100, 512)) return fail("may share");
  std::printf("ok\n");
}
"""


def test_every_key_step_is_computed_once(tmp_path):
    src, exe = tmp_path / "shares.cpp", tmp_path / "shares"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


SHARED = r"""
#include <algorithm>
#include <cstdio>
#include "prefill_shares.h"
using namespace eco;
// for each "Hq Hkv B new... cached..." line: the number of shares, from the tiles and key steps as the plan kernel finds them
int main() {
  int Hq, Hkv, B;
  while (std::scanf("%d %d %d", &Hq, &Hkv, &B) == 3) {
    int S[64], cb[64], tiles = 0, units = 0, heaviest = 0, lightest = 1 << 30, table = 0;
    for (int b = 0; b < B; ++b)
      if (std::scanf("%d", S + b) != 1) return 1;
    for (int b = 0; b < B; ++b)
      if (std::scanf("%d", cb + b) != 1) return 1;
    const int G = Hq / Hkv;
    for (int b = 0; b < B; ++b) {
      const int rows = S[b] * G, r = rows % 128;
      table = std::max(table, (S[b] + cb[b] + 63) / 64);
      for (int last = r > 0 ? r : 128; last <= rows; last += 128, ++tiles) {
        const int steps = (cb[b] + (last - 1) / G + 1 + 63) / 64;
        units += steps + kItemCost;
        heaviest = std::max(heaviest, steps);
        lightest = std::min(lightest, steps);
      }
    }
    std::printf("%d\n", may_share_steps((long long)tiles * Hkv, table, 512) ? share_wgs(tiles * Hkv, units * Hkv, heaviest, lightest, 512, B, tiles) : 0);
  }
}
"""

# the batches whose times stand at share_wgs, and some whose K and V no other tile reads
FIGURES = [((64, 8), [(366, 4351), (366, 11326)], True), ((64, 8), [(512, 16000)], True), ((40, 8), [(32, 2000)], True), ((40, 8), [(32, 16000)], True),
           ((40, 8), [(300, 5000)] * 3, True), ((8, 1), [(293, 8333)] * 5, True), ((8, 1), [(8192, 0)], True), ((8, 1), [(2000, 0)], True), ((52, 52), [(200, 4000)], True),
           ((8, 1), [(100, 3000)] * 16, True), ((64, 8), [(8, 30000)], True), ((64, 8), [(512, 0)], False), ((64, 8), [(512, 2000)], False),
           ((32, 8), [(749, 89)] * 4, False), ((40, 8), [(1024, 0)] * 4, False), ((64, 8), [(256, 2000)] * 4, False), ((64, 8), [(256, 8000)] * 8, False),
           ((8, 1), [(500, 500)] * 16, False), ((64, 8), [(2048, 0)], False), ((40, 40), [(56, 2506)] * 8, False), ((52, 52), [(100, 3000)] * 4, False),
           ((64, 8), [(1, 3000)] * 30, False), ((32, 32), [(100, 6000)] * 3, True), ((40, 8), [(20, 8000)] * 12, True)]


def test_which_batches_are_shared_out(tmp_path):
    """The batches of tests/test_gpu_prefill_shares.py are, or they would test nothing; those whose times stand beside the rule are where
    it says so."""
    from tests import test_gpu_prefill_shares as t
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(SHARED)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    calls = [(h, s, True) for h, s in t.CASES] + [((40, 8), [(8, 4000)], True)] + FIGURES
    text = "".join(f"{h[0]} {h[1]} {len(s)} " + " ".join(str(n) for n, _ in s) + " " + " ".join(str(c) for _, c in s) + "\n" for h, s, _ in calls)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split()
    assert [(c, int(n) > 0) for c, n in zip(calls, out, strict=True) if (int(n) > 0) != c[2]] == []
