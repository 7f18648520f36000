"""Decode in slices: the merge of their partial states, which is done by the slice that starts last (a few short slices: it waits for the others' states, and clears
what it has read) or is done last (long slices, or many states), eight at a time: every call finds words and counts as the first one did, whichever slices it has."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2504_18154_amd import binding
from paper_2504_18154_amd import workloads as wl
from tests.parity_util import Layer, compare, compare_lse, dev_i32, say

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (type, head size, heads, lengths, forced slices or 0): 2, 8, 9 and some 60 slices; heads whose rows a group of 16 lanes, of 32, or
# two rounds of 32 hold, whole and ragged; slices of more than four rounds; more workgroups than run at once
CASES = [("bf16", 128, (40, 8), [700, 1100, 40], 0), ("bf16", 128, (8, 1), [60000], 0), ("bf16", 128, (16, 1), [9000, 129, 3000], 0), ("bf16", 128, (8, 2), [300100], 0),
         ("f32", 64, (4, 2), [513, 64, 577], 64), ("f32", 32, (4, 2), [1025, 130], 128), ("bf16", 24, (6, 3), [700, 65], 64), ("bf16", 80, (8, 8), [600, 64, 1], 64),
         ("f32", 100, (6, 3), [577, 512], 64), ("bf16", 200, (8, 2), [640, 70], 64), ("f32", 256, (4, 2), [577, 128], 64), ("bf16", 64, (32, 8), [1300] * 40, 64),
         # counted states (long slices, or more than 96 states of short ones): all at once, and behind calls that clear theirs
         ("bf16", 128, (16, 1), [1500], 0), ("bf16", 64, (16, 1), [900, 130, 520], 64), ("f32", 64, (4, 2), [5000, 1300], 1024), ("f32", 256, (4, 2), [3000, 500], 320),
         ("bf16", 104, (24, 2), [3100, 700, 2000], 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,D,heads,lens,split", CASES, ids=[f"{c[0]}-D{c[1]}-{c[2][0]}x{c[2][1]}-B{len(c[3])}-L{max(c[3])}-{c[4]}" for c in CASES])
def test_merged_slices_call_after_call(dtype, D, heads, lens, split):
    model = wl.ModelShape("merge", heads[0], heads[1], D, 1, dtype)
    lens = np.asarray(lens, dtype=np.int32)
    say(f"decode in slices, {dtype}, head size {D}, {len(lens)} sequences up to {lens.max()} tokens, slices of {split or 'its own choice'}")
    pb = wl.prefill_batch(model, lens, 71)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    if split:
        layer.ctx.set_option(binding.OPT_DECODE_SPLIT_TOKENS, split)
    layer.append(*(wl.randn((pb.T, model.Hkv, D), dtype, s) for s in (1, 2)), pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, model.Hq, D), dtype, 3)
    ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
    out, lse = layer.decode_gpu(q, pb.block_table, lens)
    compare("decode", out, ref, dtype)
    compare_lse("decode", lse, ref_lse, dtype)
    fewer = np.maximum(1, lens // 3).astype(np.int32)
    ref2, _ = layer.decode_oracle(q, pb.block_table, fewer)
    for call in range(3):   # other slices, and the same again
        out2, _ = layer.decode_gpu(q, pb.block_table, fewer)
        compare("decode, shorter contexts", out2, ref2, dtype)
        again, lse2 = layer.decode_gpu(q, pb.block_table, lens)
        assert torch.equal(again, out) and torch.equal(lse2, lse), f"call {call} differs"
    layer.close()


@pytest.mark.gpu
@pytest.mark.parametrize("heads,n", [((16, 1), 60000), ((16, 1), 270000)], ids=["eight-wavefronts", "four-wavefronts"])
def test_rows_of_long_slices_that_are_taken_again(heads, n):
    """Long slices, two and four rows to a wavefront, and infinite V elements in two of them, one of them the newest token's: their rows are taken again key by key
    while another slice, long done, waits to merge them."""
    model = wl.ModelShape("merge", heads[0], heads[1], 128, 1, "bf16")
    lens = np.array([n], dtype=np.int32)
    say(f"decode in slices, heads {heads}, {n} tokens, infinite values")
    pb = wl.prefill_batch(model, lens, 72)
    layer = Layer(model, pb.num_blocks, 1, pb.block_table.shape[1])
    k, v = (wl.randn((n, heads[1], 128), "bf16", s) for s in (1, 2))
    for t, d in ((n // 2, 6), (n - 1, 7)):
        v[t, 0, d] = float("inf")
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q, bt, tot = wl.randn((1, heads[0], 128), "bf16", 3).cuda(), dev_i32(pb.block_table), dev_i32(lens)
    want = torch.full_like(q, float("nan"))
    layer.ctx.set_option(binding.OPT_FORCE_PLAIN, 1)
    layer.ctx.attn_decode(q, layer.kc, layer.vc, bt, tot, want, n)
    layer.ctx.set_option(binding.OPT_FORCE_PLAIN, 0)
    layer.wipe_newest(pb.block_table, lens)
    want = want.float()
    fin = torch.isfinite(want)
    assert torch.isinf(want[0, :, 6:8]).all() and int((~fin).sum()) == 2 * heads[0]
    for call in range(2):   # (the second one finds the words and counts as the first one left them)
        got = torch.full_like(q, float("nan"))
        layer.ctx.attn_decode_append(q, k[-1:].cuda(), v[-1:].cuda(), layer.kc, layer.vc, bt, tot, got, n)
        got = got.float()
        assert torch.equal(torch.isfinite(got), fin) and torch.equal(torch.isinf(got), torch.isinf(want)), f"call {call}"
        assert (got[fin] - want[fin]).abs().max() <= 2.0 ** -6   # (half a spacing of bf16, 2^-7 of |o| < 4, each, and the weights' 2^-17)
    layer.assert_cache_bit_exact()
    layer.close()


@pytest.mark.gpu
@pytest.mark.parametrize("heads,lens", [((40, 8), [2000]), ((40, 8), [700, 1100, 40]), ((8, 1), [60000]), ((40, 8), [4000] + [20] * 63)],
                         ids=["uniform", "balanced", "four-wavefronts", "cut-on-the-device"])
def test_states_that_weigh_less_than_the_smallest_normal_number(heads, lens):
    """One key of a context has all the weight, and values elsewhere, in other wavefronts' blocks (the second block) and in other slices (the last 200 tokens), are so
    large that their weight of 2^-128 counts."""
    model = wl.ModelShape("merge", heads[0], heads[1], 128, 1, "bf16")
    lens = np.asarray(lens, dtype=np.int32)
    say(f"decode in slices, heads {heads}, {len(lens)} sequences up to {lens.max()} tokens, states of weight 2^-128")
    pb = wl.prefill_batch(model, lens, 73)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v = (torch.zeros((pb.T, heads[1], 128), dtype=torch.bfloat16) for _ in range(2))
    q = torch.zeros((pb.B, heads[0], 128), dtype=torch.bfloat16)
    q[:, :, 0] = 32.0
    for first, n in zip(pb.cu_q, lens):
        if n >= 700:
            k[first, :, 0] = 31.375   # 32 x 31.375 / sqrt(128) = 88.74 = 128.03 ln 2 above the others
            v[first + 16:first + 32] = 2.0 ** 122
            v[first + n - 200:first + n] = 2.0 ** 118
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
    assert (ref[lens >= 700] > 0.4).all()
    out, lse = layer.decode_gpu(q, pb.block_table, lens)
    # half a spacing of bf16, and the weights' error: scores of 128 to 2^-17, times ln 2, and 22 bits of a number of 2^-128
    err, bound = float(np.abs(out.double().cpu().numpy() - ref).max()), float((2.0 ** -8 + 2.0 ** -16) * ref.max())
    assert err <= bound
    compare_lse("decode", lse, ref_lse, "bf16")
    layer.close()


@pytest.mark.gpu
def test_one_context_in_slices_of_several_windows():
    """52 K/V heads, one context: nine slices of some 4450 tokens in four wavefronts, whose block ids take two registers' worth one after the other."""
    model = wl.ModelShape("merge", 52, 52, 128, 1, "bf16")
    lens = np.array([40011], dtype=np.int32)
    say("decode in slices of more than 4096 tokens")
    pb = wl.prefill_batch(model, lens, 74)
    layer = Layer(model, pb.num_blocks, 1, pb.block_table.shape[1])
    k, v = (wl.randn((pb.T, 52, 128), "bf16", s, device="cuda") for s in (1, 2))
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((1, 52, 128), "bf16", 3)
    ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
    out, lse = layer.decode_gpu(q, pb.block_table, lens)
    compare("decode", out, ref, "bf16")
    compare_lse("decode", lse, ref_lse, "bf16")
    layer.wipe_newest(pb.block_table, lens)
    fused = torch.full_like(out, float("nan"))
    layer.ctx.attn_decode_append(q.cuda(), k[-1:].contiguous(), v[-1:].contiguous(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), fused, int(lens[0]))
    assert torch.equal(fused, out), "the fused append changes the result"
    layer.assert_cache_bit_exact()
    layer.close()


BOUND = r"""
#include <cstdio>
#include "decode_slices.h"
using namespace eco;
// what a context holds (slice_states in api.hip), in states per query head of a group: two workgroups per CU, or slices of 1024 tokens
int main() {
  unsigned seed = 7;
  auto rnd = [&](unsigned n) { return (seed = seed * 1664525u + 1013904223u, (unsigned)((unsigned long long)(seed >> 8) * n >> 24)); };
  for (int i = 0; i < 400000; ++i) {
    const int cu = rnd(4) ? 256 : 8 + 8 * rnd(38), Hkv = 1 + rnd(rnd(2) ? 8 : 64), B = 1 + rnd(rnd(2) ? 64 : 4096), L = 1 + rnd(1 + rnd(rnd(2) ? 4096 : 400000)), D = 8 * (1 + rnd(32)), es = rnd(2) ? 2 : 4;
    const SmallDecode s = small_decode(B, Hkv, L, cu), a = any_decode(B, Hkv, D, es, L, cu);
    const long long of_s = (long long)(s.split_tokens ? B : 1) * Hkv * s.n_split, of_a = (long long)B * Hkv * a.n_split, few = 2LL * cu;
    const long long uniform = (long long)B * Hkv * ((L + 1023) / 1024);
    if (of_s > few) return std::printf("bf16, 128: B %d, %d heads, %d tokens, %d CUs: %lld states\n", B, Hkv, L, cu, of_s), 1;
    if (of_a > (few > uniform ? few : uniform)) return std::printf("%d bytes, %d: B %d, %d heads, %d tokens, %d CUs: %lld states\n", es, D, B, Hkv, L, cu, of_a), 1;
  }
  std::printf("ok\n");
}
"""


def test_slices_states_fit_what_a_context_holds(tmp_path):
    src, exe = tmp_path / "bound.cpp", tmp_path / "bound"
    src.write_text(BOUND)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
