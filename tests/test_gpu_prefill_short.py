"""bf16 prefill behind short contexts (csrc/attn_prefill_short.hip): on the host, that each case below takes the way through the kernel
it is listed for; on the GPU, against the fp64 CPU oracle, in a cache whose unwritten slots are not numbers, with lengths at the edges of
tiles, groups of keys and cache blocks, group sizes 1 to 16, sequences without new tokens, and rows that are slices of wider
ones."""
import os
import subprocess

import numpy as np
import pytest

from paper_2504_18154_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NO, ROWS64, ROWS32, SPLIT = range(4)


def _ragged(B, most, cached, seed=71):
    rng = wl.rng_for(seed)
    return list(zip(rng.integers(0, most + 1, size=B).tolist(), rng.integers(0, cached + 1, size=B).tolist()))


# name, heads, (new, cached tokens) per sequence, way
CASES = [
    ("one-group", (40, 8), [(16, 0), (1, 31), (0, 7), (32, 0), (7, 9)], ROWS32),
    ("split-edges", (5, 1), [(93, 0), (32, 1), (33, 31), (0, 64), (64, 64), (13, 115)], SPLIT),
    ("split-long", (3, 3), [(31, 2017), (65, 1)], SPLIT),
    ("split-G16", (16, 1), [(2, 30), (4, 127), (6, 128)], SPLIT),
    ("split-more-than-a-round", (52, 52), [(300, 0)], SPLIT),
    ("split-one-and-a-half-rounds", (40, 8), [(507, 0), (63, 449), (46, 0)], SPLIT), ("split-to-1536", (8, 1), [(280, 1250), (1, 1535)] + [(200, 0)] * 10, SPLIT),
    ("rows32-many-sequences", (8, 1), _ragged(300, 40, 50), ROWS32),
    ("rows32-mha", (52, 52), _ragged(70, 20, 40), ROWS32),
    ("rows64", (40, 8), _ragged(90, 100, 60), ROWS64),
    ("rows64-mha", (52, 52), [(64, 0), (63, 1), (65, 63), (128, 2), (1, 0), (150, 31), (0, 33), (33, 96), (127, 64)] * 3, ROWS64),
    ("rows64-G8", (64, 8), [(300, 100), (399, 1), (1, 399), (257, 130)] * 6, ROWS64),
    ("too-long", (40, 8), [(20, 3000)], NO),
    # more than 16 sequences, some of them long (us by the persistent kernel / keys shared: 21.9 / 32.8, 26.8 / 29.0), and heads whose tiles do not stay
    # with one XCD, beyond 1.25 rounds of workgroups (19.4 / 22.9)
    ("17-up-to-1652", (64, 8), [(2, 200)] * 13 + [(1, 1651)] * 3 + [(51, 384)], NO), ("21-up-to-1152", (16, 4), [(53, 400)] * 20 + [(33, 1119)], NO),
    ("far-tiles-in-1.4-rounds", (52, 52), [(86, 354)] * 3 + [(87, 393)], NO),
]


def test_each_case_takes_the_way_it_is_listed_for(tmp_path):
    calls = []
    for _, heads, seqs, *_ in CASES:
        width = max((n + c + 15) // 16 for n, c in seqs)
        calls.append(f"prefill_short({len(seqs)}, {sum(n for n, _ in seqs)}, {heads[0]}, {heads[1]}, {16 * width}, 256)")
    calls += [f"prefill_short({B}, {B * n}, {heads[0]}, {heads[1]}, {(n + c + 15) // 16 * 16}, 256)" for heads, B, (n, c), _ in INFINITE]
    src, exe = tmp_path / "way.cpp", tmp_path / "way"
    src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "prefill_short.h"\nusing namespace eco;\n'
                   'int main() { for (PrefillShort w : {%s}) std::printf("%%d ", (int)w);\n'
                   # block tables of more than 2048 tokens are not for this kernel, whatever the batch
                   '  int any = 0;\n'
                   '  for (int Hkv : {1, 2, 3, 4, 8, 16, 52}) for (int G = 1; G <= 16; ++G) for (int B = 1; B <= 4096; B += B / 8 + 1) for (long T = 1; T < 200000; T += T / 4 + 1)\n'
                   '    any |= (int)prefill_short(B, T, Hkv * G, Hkv, 2064, 256);\n'
                   '  std::printf("%%d ", any); }' % ", ".join(calls))
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    got = [int(x) for x in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]
    assert got == [c[3] for c in CASES] + [c[3] for c in INFINITE] + [NO]


@pytest.mark.gpu
@pytest.mark.parametrize("case", [c for c in CASES if c[3] != NO], ids=lambda c: c[0])
def test_against_the_oracle(case):
    import torch

    from oracle import oracle as orc
    from paper_2504_18154_amd import binding
    from tests.parity_util import Layer, compare, compare_lse, dev_i32, say
    name, heads, seqs = case[:3]
    model = wl.ModelShape("short", heads[0], heads[1], 128, 1, "bf16")
    new, cached = (np.asarray(x, dtype=np.int32) for x in zip(*seqs))
    say(f"prefill, {name}, heads {heads}, {len(seqs)} sequences, {int(new.sum())} tokens behind {int(cached.sum())}")
    pb = wl.prefill_batch(model, new, 91, ctx_before=cached)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    kp, vp = (wl.randn((int(cached.sum()), model.Hkv, 128), "bf16", s) for s in (1, 2))
    layer.append(kp, vp, wl.cu_from_lengths(cached), np.zeros(pb.B, np.int32), pb.block_table)
    q = wl.randn((pb.T, model.Hq, 128), "bf16", 3)
    layer.append(*(wl.randn((pb.T, model.Hkv, 128), "bf16", s) for s in (4, 5)), pb.cu_q, pb.ctx_before, pb.block_table)
    out, lse = layer.prefill_gpu(q, pb.cu_q, pb.ctx_before, pb.block_table)
    rows = np.sort(wl.rng_for(92).choice(pb.T, size=min(pb.T, 400), replace=False)).astype(np.int64)
    seq = np.searchsorted(pb.cu_q, rows, side="right") - 1
    start = np.searchsorted(seq, np.arange(pb.B + 1), side="left").astype(np.int32)
    pos = pb.ctx_before[seq] + (rows - pb.cu_q[seq])
    ref, ref_lse = orc.attn_rows(layer.shape, wl.to_bits(q), layer.okc, layer.ovc, pb.block_table, start, rows.astype(np.int32), pos.astype(np.int32))
    compare("prefill", out, ref, "bf16", rows=rows)
    compare_lse("prefill", lse, ref_lse, "bf16", rows=rows, bf16_row_sum=True)
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    # rows that are slices of a wider one, without log-sum-exps, recorded and replayed: the same bits
    cu, cb, bt = dev_i32(pb.cu_q), dev_i32(pb.ctx_before), dev_i32(pb.block_table)
    wide = torch.full((pb.T, model.Hq + 2 * model.Hkv, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide[:, :model.Hq] = q.cuda()
    o = torch.full_like(out, float("nan"))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer.ctx.attn_prefill_strided(wide[:, :model.Hq], layer.kc, layer.vc, cu, cb, bt, o, None, max_q_len=int(new.max()))
    for _ in range(3):
        o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, out)
    # the same where the layers of a step would share a list of tiles
    layer.ctx.set_option(binding.OPT_PREFILL_REUSE_PLAN, 1)
    o.fill_(float("nan"))
    layer.ctx.attn_prefill(q.cuda(), layer.kc, layer.vc, cu, cb, bt, o, None, max_q_len=int(new.max()))
    assert torch.equal(o, out)
    layer.close()


# heads, sequences, (new, cached) tokens of each, way
INFINITE = [((40, 8), 1, (8, 1000), SPLIT), ((8, 1), 200, (8, 60), ROWS32), ((64, 8), 50, (64, 100), ROWS64)]


@pytest.mark.gpu
@pytest.mark.parametrize("heads,B,tokens,way", INFINITE, ids=["split", "rows32", "rows64"])
def test_keys_of_minus_infinity_weigh_nothing(heads, B, tokens, way):
    """Also where they fill a walk's first groups of 32 keys, or all the groups of one of four wavefronts but the last."""
    import torch

    from tests.parity_util import Layer, dev_i32, say
    (new, cached), (Hq, Hkv) = tokens, heads
    n = new + cached
    model = wl.ModelShape("short", Hq, Hkv, 128, 1, "bf16")
    say(f"prefill, keys of minus infinity, heads {heads}, {B} x {new} tokens behind {cached}")
    pb = wl.prefill_batch(model, np.full(B, new, np.int32), 93, ctx_before=np.full(B, cached, np.int32))
    layer = Layer(model, pb.num_blocks, B, pb.block_table.shape[1], oracle_cache=False)
    dead = torch.zeros(n, dtype=torch.bool)
    dead[:40] = True
    for g in range(1, cached // 32, 4):
        dead[32 * g:32 * g + 32] = True
    k = torch.zeros((n, Hkv, 128), dtype=torch.bfloat16)
    k[dead, :, 0] = -float("inf")
    v = wl.randn((n, Hkv, 128), "bf16", 6)
    layer.ctx.kv_append(layer.kc, layer.vc, k.repeat(B, 1, 1).cuda(), v.repeat(B, 1, 1).cuda(), dev_i32(np.arange(B + 1) * n), dev_i32(np.zeros(B)), dev_i32(pb.block_table))
    q = torch.zeros((pb.T, Hq, 128), dtype=torch.bfloat16)
    q[:, :, 0] = 1.0
    out, lse = layer.prefill_gpu(q, pb.cu_q, pb.ctx_before, pb.block_table)
    out, lse = out.view(B, new, Hq, 128).double().cpu(), lse.view(B, new, Hq).double().cpu()
    # equal weights on all other keys: running means of V
    for i in range(new):
        keys = torch.arange(cached + i + 1)[~dead[:cached + i + 1]]
        ref = v[keys].double().mean(0).repeat_interleave(Hq // Hkv, dim=0)
        assert (out[:, i] - ref).abs().max() <= 1e-2
        assert (lse[:, i] - np.log(len(keys))).abs().max() <= 1e-3
    layer.close()


@pytest.mark.gpu
def test_a_shared_tile_list_does_not_outlive_a_batch_without_one():
    """Calls of one step share their list of tiles (ECOSERVE_OPT_PREFILL_REUSE_PLAN).  A call that needs none comes between two that name the
    same arrays, whose contents have changed with the batch: the second makes its own."""
    import torch

    from paper_2504_18154_amd import binding
    from tests.parity_util import Layer, compare, dev_i32, say
    model = wl.ModelShape("short", 40, 8, 128, 1, "bf16")
    lens = np.asarray([700, 1500], dtype=np.int32)
    say("prefill, long, short and long again with a list that is shared")
    pb = wl.prefill_batch(model, np.full(2, 1500, np.int32), 95)
    layer = Layer(model, pb.num_blocks, 2, pb.block_table.shape[1])
    layer.ctx.set_option(binding.OPT_PREFILL_REUSE_PLAN, 1)
    cu, cb, wide = dev_i32(np.r_[0, 0, 0]), dev_i32([0, 0]), dev_i32(np.pad(pb.block_table, ((0, 0), (0, 40)), constant_values=-1))
    narrow = wide[:, :2].contiguous()
    for new, table in ((lens, wide), (np.asarray([20, 11], np.int32), narrow), (lens[::-1].copy(), wide)):
        cu.copy_(dev_i32(wl.cu_from_lengths(new)))
        T = int(new.sum())
        k, v = (wl.randn((T, 8, 128), "bf16", s + T) for s in (1, 2))
        layer.append(k, v, wl.cu_from_lengths(new), np.zeros(2, np.int32), pb.block_table)
        q = wl.randn((T, 40, 128), "bf16", 3)
        out = torch.full((T, 40, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        for _ in range(2):
            layer.ctx.attn_prefill(q.cuda(), layer.kc, layer.vc, cu, cb, table, out, None, max_q_len=int(new.max()))
        ref, _ = layer.prefill_oracle(q, wl.cu_from_lengths(new), np.zeros(2, np.int32), pb.block_table)
        compare(f"{new.tolist()} tokens", out, ref, "bf16")
    layer.close()
