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
