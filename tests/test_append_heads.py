"""csrc/append_heads.h, the rule by which the tiled append kernel is picked: on the host, that each case below takes the instance it
is listed for; on the GPU, that the instance fills the cache as the oracle does, bit for bit, with ragged sequences behind cached
tokens that end within a block."""
import os
import subprocess

import numpy as np
import pytest

from paper_2504_18154_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# dtype, head size, K/V heads, sequences, most new tokens of one: heads per workgroup, loads at once (256 CUs)
CASES = [("bf16", 128, 8, 16, 400, 1, True), ("bf16", 128, 8, 16, 600, 2, False),        # around eight workgroups per CU
         ("bf16", 128, 8, 128, 240, 2, False), ("bf16", 128, 8, 128, 272, 4, False),     # around forty heads' blocks per CU
         ("bf16", 128, 3, 500, 9, 1, False), ("bf16", 64, 4, 500, 1, 2, False), ("bf16", 64, 4, 640, 9, 4, False), ("bf16", 256, 4, 40, 400, 2, False),
         ("f32", 128, 4, 1280, 3, 4, False), ("f32", 256, 4, 20, 100, 1, False), ("f32", 256, 4, 1200, 12, 4, False),  # the last: raised LDS limit
         ("f32", 256, 2, 2400, 12, 1, False), ("f32", 64, 4, 6, 200, 1, True)]
IDS = [f"{c[0]}-{c[1]}-{c[2]}heads-B{c[3]}-{c[4]}" for c in CASES]


def _new_tokens(case):
    new = wl.rng_for(61).integers(0, case[4] + 1, size=case[3])
    new[:2] = case[4]
    return new.astype(np.int32)


def test_each_case_takes_the_instance_it_is_listed_for(tmp_path):
    calls = ", ".join(f"append_heads({int(_new_tokens(c).sum())}, {c[3]}, {c[2]}, {c[1] * (2 if c[0] == 'bf16' else 4)}, 256)" for c in CASES)
    src, exe = tmp_path / "heads.cpp", tmp_path / "heads"
    src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "append_heads.h"\nusing namespace eco;\nint main() { for (AppendHeads h : {%s}) std::printf("%%d %%d\\n", h.heads, h.at_once); }' % calls)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    assert [(int(a), int(b)) for a, b in zip(out[::2], out[1::2])] == [(c[5], int(c[6])) for c in CASES]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_append_is_bit_exact(case):
    from tests.parity_util import Layer, say
    dtype, D, Hkv, B = case[:4]
    model = wl.ModelShape("append", Hkv, Hkv, D, 1, dtype)
    new = _new_tokens(case)
    first = wl.rng_for(62).integers(0, 19, size=B).astype(np.int32)
    say(f"append, {dtype}, head size {D}, {Hkv} K/V heads: {int(first.sum())} then {int(new.sum())} tokens of {B} sequences")
    pb = wl.prefill_batch(model, np.maximum(first + new, 1), 63)
    layer = Layer(model, pb.num_blocks, B, pb.block_table.shape[1])
    for seed, n, before in ((1, first, np.zeros_like(first)), (3, new, first)):
        k, v = (wl.randn((int(n.sum()), Hkv, D), dtype, s) for s in (seed, seed + 1))
        layer.append(k, v, wl.cu_from_lengths(n), before, pb.block_table, max_new_len=max(2, int(n.max())))
    layer.assert_cache_bit_exact()
    layer.close()
