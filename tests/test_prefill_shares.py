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
  if (share_wgs(32, 32 * 5, 2, 2, 512) || share_wgs(512, 512 * 53, 50, 50, 512) || share_wgs(1280, 1280 * 20, 32, 1, 512)) return fail("shares");
  if (!share_wgs(8, 8 * 253, 250, 250, 512) || !share_wgs(584, 584LL * 171, 200, 103, 512)) return fail("no shares");
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
