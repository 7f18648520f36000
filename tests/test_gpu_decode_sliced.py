"""Decode of whole contexts with the longer ones cut, on the device and by all lengths of the batch: at the edges of its slices, groups and ranks, with
contexts that are empty, alone among short ones or all alike; and what the persistent kernel keeps, larger batches."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2504_18154_amd import binding
from paper_2504_18154_amd import workloads as wl
from tests.parity_util import Layer, compare, compare_lse, dev_i32, say

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _mix(seed, n, lo, hi):
    return np.random.default_rng(seed).integers(lo, hi, size=n)


SLICED = [((40, 8), np.r_[4000, [20] * 63]),                                       # one is cut, the rest are short
          ((40, 8), np.r_[[384] * 20, 385, 400, 383, 768, 769, [1500] * 20]),      # multiples of the shortest slice, and a token on either side
          ((64, 8), np.r_[0, _mix(1, 62, 1, 3000), 0, 0, _mix(2, 40, 1, 600), 2999, 16, 17, 0]),   # two groups, empty ones among them
          ((8, 1), _mix(3, 200, 1, 4000)), ((16, 1), _mix(4, 256, 700, 2400)),     # four groups; sixteen heads to a group
          ((52, 52), np.array([40, 900, 2500, 700, 1800, 300, 3000])), ((5, 5), _mix(5, 65, 1400, 1700))]
# (empty sequences first, last and in a row; one context of some 840 pieces, whose states the merge takes 64 at a time)
PERSISTENT = [((40, 8), _mix(6, 257, 100, 1800)), ((52, 52), _mix(7, 40, 900, 2000)), ((8, 1), np.r_[0, 0, 60000, 0, _mix(8, 130, 1, 100), 0, 0, 0, 16, _mix(9, 130, 1, 100), 17, 0]),
              ((64, 8), np.r_[_mix(10, 150, 1, 60), 0, 4000, 0, 0, _mix(11, 150, 1, 60), 0])]


@pytest.mark.gpu
@pytest.mark.parametrize("heads,lens", SLICED + PERSISTENT, ids=[f"{h[0]}x{h[1]}-B{len(n)}-L{max(n)}" for h, n in SLICED + PERSISTENT])
def test_batches_of_long_contexts(heads, lens):
    model = wl.ModelShape("sliced", heads[0], heads[1], 128, 1, "bf16")
    lens = np.asarray(lens, dtype=np.int32)
    say(f"decode, heads {heads}, {len(lens)} sequences up to {lens.max()} tokens")
    pb = wl.prefill_batch(model, np.maximum(lens, 1), 61)
    layer = Layer(model, pb.num_blocks, len(lens), pb.block_table.shape[1])
    k, v = (wl.randn((int(lens.sum()), model.Hkv, 128), "bf16", s) for s in (1, 2))
    layer.append(k, v, wl.cu_from_lengths(lens), np.zeros_like(lens), pb.block_table)
    q = wl.randn((len(lens), model.Hq, 128), "bf16", 3)
    live = np.flatnonzero(lens > 0)
    ref, ref_lse = layer.decode_oracle(q[live], pb.block_table[live], lens[live])
    out, lse = layer.decode_gpu(q, pb.block_table, lens)
    compare("decode", out[live], ref, "bf16")
    compare_lse("decode", lse[live], ref_lse, "bf16")
    assert torch.isnan(out[lens == 0].float()).all()   # (as the caller left them)
    fewer = np.where(lens > 2, lens // 2, lens).astype(np.int32)
    layer.decode_gpu(q, pb.block_table, fewer)         # (other slices in between)
    again, lse2 = layer.decode_gpu(q, pb.block_table, lens)
    assert torch.equal(again[live], out[live]) and torch.equal(lse2[live], lse[live]), "a second call differs"
    last = torch.as_tensor(np.maximum(np.cumsum(lens) - 1, 0), dtype=torch.long)
    fused, fused_lse = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
    layer.wipe_newest(pb.block_table[live], lens[live])
    layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens),
                                 fused, int(lens.max()), fused_lse)
    no = torch.full_like(out, float("nan"))
    assert binding.attn_decode_noalloc(layer.ctx.layout, q.cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), no, int(lens.max())) == binding.OK
    torch.cuda.synchronize()
    assert torch.equal(fused[live], out[live]) and torch.equal(fused_lse[live], lse[live]), "the fused append changes the result"
    assert torch.equal(no[live], out[live]), "the call without a context differs"
    layer.assert_cache_bit_exact()
    layer.close()


@pytest.mark.gpu
def test_infinite_values_in_contexts_that_are_cut():
    """Infinite V elements, one in the token that the fused append brings: infinite there, elsewhere as the plain kernels have it."""
    model = wl.ModelShape("sliced", 40, 8, 128, 1, "bf16")
    lens = np.r_[3000, 2999, [700] * 60].astype(np.int32)
    pb = wl.prefill_batch(model, lens, 62)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v = (wl.randn((pb.T, 8, 128), "bf16", s) for s in (1, 2))
    for t, g, d in ((33, 1, 5), (1500, 1, 6), (2999, 2, 7)):
        v[t, g, d] = float("inf")
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, 40, 128), "bf16", 3)
    last = torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)
    res = []
    for plain in (0, 1):
        layer.ctx.set_option(binding.OPT_FORCE_PLAIN, plain)
        layer.wipe_newest(pb.block_table, lens)
        out = torch.full((pb.B, 40, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), out, int(lens.max()))
        torch.cuda.synchronize()
        layer.assert_cache_bit_exact()
        res.append(out.float())
    got, want = res
    fin = torch.isfinite(want)
    assert torch.isinf(want[0, 5:10, 5:7]).all() and torch.isinf(want[0, 10:15, 7]).all() and int((~fin).sum()) == 15
    assert torch.equal(torch.isfinite(got), fin) and torch.equal(torch.isinf(got), torch.isinf(want))
    assert (got[fin] - want[fin]).abs().max() <= 2.0 ** -6   # half a spacing of bf16 (2^-7 of |o| < 4) each, and the weights' 2^-17
    layer.close()


@pytest.mark.gpu
@pytest.mark.parametrize("heads,lens", [((40, 8), np.r_[3000, 1, 0, 2999, _mix(12, 60, 300, 900)]), ((16, 1), np.r_[6000, 40, 700]), ((8, 1), np.r_[20000]), ((40, 8), np.r_[777]),
                                        ((40, 8), np.r_[2000, 128, 129, 0, 1024, 16, 700, 1])], ids=["cut-on-the-device", "many-states", "long-slices", "arrival-words", "balanced"])
def test_graphs_of_decode_in_slices(heads, lens):
    """A recorded step, replayed with other lengths and queries and the program's own calls on the context in between: each replay as the call."""
    model = wl.ModelShape("sliced", heads[0], heads[1], 128, 1, "bf16")
    lens = np.asarray(lens, dtype=np.int32)
    say(f"graph of decode in slices, heads {heads}, {len(lens)} sequences up to {lens.max()} tokens")
    pb = wl.prefill_batch(model, np.maximum(lens, 1), 63)
    layer = Layer(model, pb.num_blocks, len(lens), pb.block_table.shape[1], oracle_cache=False)
    for c, s in ((layer.kc, 4), (layer.vc, 5)):
        c.copy_(wl.randn(c.shape, "bf16", s, device="cuda"))
    q, kn, vn = (wl.randn((len(lens), h, 128), "bf16", s, device="cuda") for h, s in ((heads[0], 1), (heads[1], 2), (heads[1], 3)))
    bt, tot, out, bound = dev_i32(pb.block_table), dev_i32(lens), torch.zeros_like(q), int(lens.max())

    def step():
        for _ in range(2):
            layer.ctx.attn_decode_append(q, kn, vn, layer.kc, layer.vc, bt, tot, out, bound)

    step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for r in range(4):
        q.copy_(wl.randn(q.shape, "bf16", 70 + r, device="cuda"))
        tot.copy_(dev_i32(np.maximum(lens - 37 * r, np.minimum(lens, 1))))
        out.fill_(float("nan"))
        step()
        torch.cuda.synchronize()
        want = out.clone()
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        live = (tot > 0).cpu().numpy()
        assert torch.isfinite(want[live].float()).all() and torch.equal(out[live], want[live]), f"replay {r}"
    layer.close()


RULE = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "decode_slices.h"
using namespace eco;
// one line per batch: "B Hkv bound adaptive", answered by the kernel that takes it; then, over random batches, what the kernel makes of the lengths
int main() {
  int B, Hkv, bound, adaptive;
  while (std::scanf("%d %d %d %d", &B, &Hkv, &bound, &adaptive) == 4)
    std::printf("%s\n", decode_short(B, Hkv, bound, 256) ? "whole" : small_decode(B, Hkv, bound, 256).n_split ? "small"
                         : decode_sliced(B, Hkv, 256) && !(adaptive && adaptive_stream(B, Hkv, bound, 256)) ? "sliced" : "persistent");
  unsigned seed = 99;
  auto rnd = [&](unsigned n) { return (seed = seed * 1664525u + 1013904223u, (unsigned)((unsigned long long)(seed >> 8) * n >> 24)); };
  for (int i = 0; i < 30000; ++i) {
    const int heads[] = {1, 2, 3, 4, 5, 8, 16, 52, 300, 2000};
    Hkv = heads[rnd(10)];
    B = 1 + rnd(256);
    if (!decode_sliced(B, Hkv, 256)) continue;
    const int W = 4, most = 1 + rnd(rnd(3) ? 400 : rnd(2) ? 40000 : 2000000), shape = rnd(4), max_full = sliced_most_full(B, Hkv, 256);
    std::vector<int> nb(B);
    long long sum = 0;
    for (int b = 0; b < B; ++b) sum += nb[b] = shape == 0 ? rnd(most + 1) : shape == 1 ? (rnd(2) ? 0 : rnd(most + 1)) : shape == 2 ? (b ? rnd(4) : most) : most;
    if (sum > 0x7fffffff) continue;
    const SlicedContexts c = sliced_contexts((int)sum, max_full, W);
    if (c.blocks % W || c.blocks < 24) return std::printf("%d blocks\n", c.blocks), 1;
    const int groups = (B + 63) / 64, per_group = (B + groups - 1) / groups;
    long long before = 0, slots = 0;
    for (int g = 0; g < groups; ++g) {
      long long full = 0;
      int have = 0;
      for (int b = g; b < B; b += groups, ++have) {
        const int f = c.full(nb[b]), left = nb[b] - f * c.blocks;
        if (f < 0 || (nb[b] && left <= 0) || left > 2 * c.blocks || c.size_class(left) < 0 || c.size_class(left) > 15) return std::printf("%d of %d blocks\n", nb[b], c.blocks), 1;
        full += f;
        slots += f ? f + 1 : 0;
      }
      if (have > 64 || have != (B - g + groups - 1) / groups || have > per_group) return std::printf("group %d of %d: %d\n", g, groups, have), 1;
      if (full > max_full) return std::printf("%lld whole slices of %d\n", full, max_full), 1;  // (the grid has per_group + max_full ranks)
      before += full;
    }
    if (before > max_full || slots > 2LL * max_full || slots * Hkv > 6LL * 256) return std::printf("%lld slots\n", slots), 1;
  }
  std::printf("ok\n");
}
"""


def test_slices_slots_and_the_kernels_of_the_batches(tmp_path):
    """Every context is covered once, whole slices and slots fit the grid and what a context holds; and which kernel takes the batches above, and
    those of the tests and of the benchmark."""
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(RULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    calls = [(len(n), h[1], int(max(n)), 0) for h, n in SLICED + PERSISTENT]
    calls += [(62, 8, 3000, 0), (128, 8, 4096, 1), (256, 8, 4096, 0), (200, 8, 9000, 0), (160, 8, 4000, 1)]
    calls += [(257, 8, 4096, 0), (1024, 8, 1700, 0), (256, 8, 4096, 1), (200, 8, 9000, 1), (160, 8, 4001, 1), (1, 8, 80000, 0), (1, 1, 4000000, 1)]
    want = ["sliced"] * len(SLICED) + ["persistent"] * len(PERSISTENT) + ["sliced"] * 5 + ["persistent"] * 5 + ["small"] * 2
    r = subprocess.run([str(exe)], input="".join(f"{b} {h} {n} {a}\n" for b, h, n, a in calls), capture_output=True, text=True)
    got = r.stdout.split()
    assert got[len(want):] == ["ok"], r.stdout[-300:]
    assert got[:len(want)] == want, [(c, g, w) for c, g, w in zip(calls, got, want) if g != w]
