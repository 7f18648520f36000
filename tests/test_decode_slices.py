"""csrc/decode_slices.h, the arithmetic by which the small-batch decode kernel cuts a context and reads the block table,
compiled for the host: the slices cover the context once, and the block table entries read by all wavefronts of all slices
are those of the sequence's blocks, each once, and none behind them (such an entry may not even be backed by memory)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "decode_slices.h"
int main() {
  const int lens[] = {0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1024, 1025, 2048, 4095, 4096, 4097, 9000};
  for (int split : {64, 192, 256, 512, 1024, 4096})
    for (int waves : {4, 8})
      for (int L : lens)
        for (int bound : {L, 1, 700, 1024, 20000}) {  // the caller's bound on the length: right, too low, generous
          const int grid = bound > 0 ? (bound + split - 1) / split : 1;
          const int blocks = (L + 15) / 16;
          std::vector<int> read(blocks, 0);
          int next = 0;
          for (int sp = 0; sp < grid; ++sp) {
            const eco::Slice s = eco::decode_slice(L, split, grid, sp);
            if (sp >= s.n) continue;
            if (s.t0 != next || s.t1 <= s.t0 || s.t0 % 16 != 0) return std::printf("slice %d of %d tokens: [%d, %d)\n", sp, L, s.t0, s.t1), 1;
            next = s.t1;
            for (int w = 0; w < waves; ++w) {
              const eco::WaveBlocks b = eco::wave_blocks(s.t0, s.t1, w, waves);
              for (int i = 0; i < b.n; ++i) {
                const int e = b.first + b.step * i;
                if (e < 0 || e >= blocks) return std::printf("%d tokens: entry %d of %d is read\n", L, e, blocks), 1;
                ++read[e];
              }
            }
          }
          if (next != L) return std::printf("%d tokens: %d covered\n", L, next), 1;
          for (int e = 0; e < blocks; ++e)
            if (read[e] != 1) return std::printf("%d tokens: entry %d is read %d times\n", L, e, read[e]), 1;
        }
  std::printf("ok\n");
}
"""


def test_slices_and_block_table_entries(tmp_path):
    src, exe = tmp_path / "slices.cpp", tmp_path / "slices"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


RULE = r"""
#include <cstdio>
#include <cstdlib>
#include "decode_slices.h"
using namespace eco;
// the balanced slices of the contexts `len`, as the kernel finds them; false: they do not cover every context once
static bool covers(const int* len, int B, int Hkv, int slots, int W) {
  int longest = 0, sum = 0, n[64];
  for (int b = 0; b < B; ++b) {
    const int nb = (len[b] + 15) >> 4;
    longest = nb > longest ? nb : longest;
    sum += nb;
  }
  int st = first_balanced_slice(longest, sum, Hkv, slots, W), all;
  for (;; st = next_balanced_slice(st, W)) {
    all = 0;
    for (int b = 0; b < B; ++b) all += n[b] = balanced_slices_of((len[b] + 15) >> 4, st);
    if (st >= longest || all <= slots) break;
  }
  if (all > slots || st <= 0) return false;
  for (int b = 0; b < B; ++b) {
    int next = 0;
    for (int sp = 0; sp < n[b]; ++sp) {
      const Slice s = decode_slice(len[b], st * 16, n[b], sp);
      if (s.n != n[b] || s.t0 != next || s.t1 <= s.t0) return false;
      next = s.t1;
    }
    if (next != len[b]) return false;
  }
  return true;
}
// for each "B Hkv longest bound len..." line: the rule's answer, and whether its balanced slices cover the contexts; then random ones
int main() {
  int B, Hkv, bound, len[64];
  while (std::scanf("%d %d %d", &B, &Hkv, &bound) == 3) {
    for (int b = 0; b < B; ++b) {
      int x;
      if (std::scanf("%d", &x) != 1) return 1;
      if (b < 64) len[b] = x;
    }
    const SmallDecode d = small_decode(B, Hkv, bound, 256);
    const int W = d.n_split == 256 / Hkv ? 8 : 4;
    std::printf("%s\n", decode_short(B, Hkv, bound, 256) ? "whole" : d.n_split == 0 ? (decode_sliced(B, Hkv, 256) ? "sliced" : "persistent") : d.split_tokens > 0 ? "uniform" : !covers(len, B, Hkv, d.n_split, W) ? "wrong" : W == 8 ? "8" : "4");
  }
  unsigned seed = 12345;
  auto rnd = [&](unsigned n) { return (seed = seed * 1664525u + 1013904223u, (unsigned)((unsigned long long)(seed >> 8) * n >> 24)); };
  int balanced = 0;
  for (int i = 0; i < 200000; ++i) {
    const int heads[] = {1, 2, 3, 4, 5, 8, 16, 52};
    Hkv = heads[rnd(8)];
    B = 2 + rnd(63);
    const int most = 1 + rnd(rnd(3) ? 3000 : 600000 / (B * Hkv)), shape = rnd(4);
    for (int b = 0; b < B; ++b) len[b] = shape == 0 ? rnd(most + 1) : shape == 1 ? (rnd(2) ? 0 : rnd(most + 1)) : shape == 2 ? (b ? rnd(40) : most) : most;
    bound = most + (rnd(2) ? 0 : rnd(2000));
    const SmallDecode d = small_decode(B, Hkv, bound, 256);
    if (decode_short(B, Hkv, bound, 256) || d.n_split == 0 || d.split_tokens > 0) continue;
    ++balanced;
    if (!covers(len, B, Hkv, d.n_split, d.n_split == 256 / Hkv ? 8 : 4)) return std::printf("B %d, %d heads, up to %d tokens: not covered\n", B, Hkv, most), 1;
  }
  std::printf("%s\n", balanced > 20000 ? "covered" : "too few");
}
"""

# the paths that the batches of the GPU tests are there for: at the longest context's length, and with the looser bound
PATHS = {"RAGGED": ["uniform uniform", "8 8", "8 8", "uniform uniform", "8 8", "uniform uniform", "8 8", "uniform uniform", "4 sliced", "4 sliced"]}


def test_paths_of_the_batches_of_the_gpu_tests_and_their_balanced_slices(tmp_path):
    from tests import test_gpu_small_decode as t
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(RULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    calls, want = [], []
    for (heads, lens), path in zip(t.RAGGED, PATHS["RAGGED"], strict=True):
        for above, p in zip((0, 3000), path.split()):
            calls.append((heads[1], lens, max(lens) + above))
            want.append(p)
    for heads, lens, above, waves in t.BALANCED:
        calls += [(heads[1], lens, max(lens)), (heads[1], lens, max(lens) + above)]
        want += [str(waves)] * 2
    # the short ones in slices, with the bounds that the tests hand over
    calls += [(heads[1], lens, max(lens)) for heads, lens in t.CASES + t.WHOLE] + [(8, [9000, 20], 600), (8, [700, 40], 700), (2, [320], 1000), (2, [320] * 90, 1000)]
    want += ["uniform"] * len(t.CASES) + ["whole"] * len(t.WHOLE) + ["uniform"] * 4
    # many short ones that the persistent kernel has with a loose bound (test_gpu_parity.py), and the batches of test_gpu_full_configs.py, test_zz_no_alloc.py and bench.py
    calls += [(8, [300] * 800, 300), (8, [300] * 800, 1000), (8, [100] * 800, 1000), (8, [3000] * 96, 3000), (8, [4096] * 128, 4096), (8, [4096] * 256, 4096), (52, [700] * 7, 700),
              (8, [9000] * 200, 9000)]
    want += ["whole", "persistent", "persistent", "sliced", "sliced", "sliced", "whole", "sliced"]
    # batches with empty sequences, and those without a context
    calls += [(8, [1500] + [0] * 39, 1500), (8, [1500] + [0] * 47, 1500), (8, [34000, 40], 34000), (8, [60000, 40], 60000), (8, [8000, 40], 8000)]
    want += ["4", "sliced", "8", "sliced", "8"]
    text = "\n".join(f"{len(n)} {h} {bound} " + " ".join(map(str, n)) for h, n, bound in calls) + "\n"
    r = subprocess.run([str(exe)], input=text, capture_output=True, text=True)
    got = r.stdout.split("\n")
    assert got[len(want):] == ["covered", ""], r.stdout[-300:]
    assert got[:len(want)] == want, [(c[0], len(c[1]), c[2], g, w) for c, g, w in zip(calls, got, want) if g != w]


SLOTS = r"""
#include <cstdio>
#include "decode_slices.h"
using namespace eco;
// partial states per CU and query head of a group, of a device of `cu`: two for what (bf16, 128) cuts and one for what other layouts do, unless in slices of 1024 tokens; six for
// what is cut on the device
int main() {
  for (int cu : {256, 304, 64, 7})
    for (int Hkv : {1, 2, 3, 4, 5, 8, 16, 52, 256, 300})
      for (int B = 1; B <= 600; B += B / 8 + 1)
        for (int L = 1; L < 2000000; L += L / 12 + 1) {
          const long long pairs = (long long)B * Hkv;
          const SmallDecode d = small_decode(B, Hkv, L, cu);
          if (d.n_split > 1 && (d.split_tokens ? pairs : Hkv) * d.n_split > 2 * cu) return std::printf("%d x %d on %d heads: %d slices of %d\n", B, L, Hkv, d.n_split, d.split_tokens), 1;
          if (2LL * sliced_most_full(B, Hkv, cu) * Hkv > 6 * cu) return std::printf("%d on %d heads: %d whole slices\n", B, Hkv, sliced_most_full(B, Hkv, cu)), 1;
          for (int D : {24, 64, 200, 256}) {
            const SmallDecode a = any_decode(B, Hkv, D, D == 64 ? 4 : 2, L, cu);
            if (a.n_split > 1 && pairs * a.n_split > cu && a.split_tokens != 1024) return std::printf("head size %d, %d x %d on %d heads: %d slices of %d\n", D, B, L, Hkv, a.n_split, a.split_tokens), 1;
          }
        }
  std::printf("ok\n");
}
"""


def test_the_states_of_what_is_cut_fit_what_a_context_holds(tmp_path):
    src, exe = tmp_path / "slots.cpp", tmp_path / "slots"
    src.write_text(SLOTS)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


ANY = r"""
#include <cstdio>
#include "decode_slices.h"
using namespace eco;
int main() {
  // head sizes, lengths and batches of every layout: slices of whole rounds, never longer than 1024 tokens (a wavefront's 64 block ids),
  // as many as the context has, and no more than one workgroup per CU where the uniform ones would not be more either
  for (int es : {2, 4})
    for (int D = es == 2 ? 8 : 4; D <= 256; D += es == 2 ? 8 : 4)
      for (int pairs : {1, 2, 3, 8, 40, 64, 128, 200, 256, 300, 5000})
        for (int L = 1; L < 40000; L += L / 16 + 1) {
          if (D == 128 && es == 2) continue;
          const SmallDecode d = any_decode(pairs, 1, D, es, L, 256);
          const int u = decode_any_split_tokens(pairs, 1, L, 256), n_u = (L + u - 1) / u;
          if (d.split_tokens < 64 || d.split_tokens > 1024 || d.split_tokens % (16 * decode_wavefronts(D, es)) || d.n_split != (L + d.split_tokens - 1) / d.split_tokens ||
              (pairs * d.n_split > 256 && d.n_split > n_u))
            return std::printf("%d bytes, head size %d, %d pairs, %d tokens: %d of %d\n", es, D, pairs, L, d.n_split, d.split_tokens), 1;
        }
  // where cutting a context costs more than it saves
  struct { int pairs, D, es, L, tokens; } at[] = {{2, 32, 2, 2000, 256}, {4, 96, 2, 4000, 256}, {128, 128, 4, 300, 1024}, {128, 96, 4, 300, 1024}, {1, 256, 2, 1100, 256}};
  for (auto& c : at)
    if (any_decode(c.pairs, 1, c.D, c.es, c.L, 256).split_tokens != c.tokens) return std::printf("head size %d, %d tokens\n", c.D, c.L), 1;
  std::printf("ok\n");
}
"""


def test_slices_of_other_layouts(tmp_path):
    src, exe = tmp_path / "any.cpp", tmp_path / "any"
    src.write_text(ANY)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
