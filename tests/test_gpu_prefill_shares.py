"""bf16 prefill of few query tiles behind long contexts, whose key steps are shared out among the workgroups (a tile's pieces
are merged by whichever workgroup is done last): against the fp64 CPU oracle, called twice, with lengths at the edges of
tiles, key steps and cache blocks, group sizes 1 to 16, pieces from two to some thirty per tile."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2504_18154_amd import binding
from paper_2504_18154_amd import workloads as wl
from tests.parity_util import Layer, compare, compare_lse, dev_i32, say

pytestmark = pytest.mark.gpu

# heads, (new tokens, cached tokens) per sequence (the first: in the kernel for short contexts, whose wavefronts share the keys instead)
CASES = [((40, 8), [(32, 2000)]), ((40, 8), [(32, 2100)]), ((40, 8), [(1, 6000), (300, 5001), (0, 700), (26, 4095)]), ((64, 8), [(16, 4096), (17, 4097), (47, 3999)]),
         ((16, 1), [(9, 9000)]), ((5, 1), [(120, 15), (1, 7000), (64, 3000)]), ((3, 3), [(129, 2500), (63, 2559), (200, 2000)]),
         ((52, 52), [(100, 1500)]), ((8, 1), [(2500, 0), (333, 64)]), ((8, 1), [(60, 30000)])]


@pytest.mark.parametrize("heads,seqs", CASES, ids=[f"{h[0]}x{h[1]}-" + "-".join(f"{n}+{c}" for n, c in s) for h, s in CASES])
def test_shared_key_steps(heads, seqs):
    model = wl.ModelShape("shares", heads[0], heads[1], 128, 1, "bf16")
    new, cached = (np.asarray(x, dtype=np.int32) for x in zip(*seqs))
    say(f"prefill, heads {heads}, new + cached tokens {seqs}")
    pb = wl.prefill_batch(model, new, 91, ctx_before=cached)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    kp, vp = (wl.randn((int(cached.sum()), model.Hkv, 128), "bf16", s) for s in (1, 2))
    layer.append(kp, vp, wl.cu_from_lengths(cached), np.zeros(pb.B, np.int32), pb.block_table)
    q = wl.randn((pb.T, model.Hq, 128), "bf16", 3)
    layer.append(*(wl.randn((pb.T, model.Hkv, 128), "bf16", s) for s in (4, 5)), pb.cu_q, pb.ctx_before, pb.block_table)
    out, lse = layer.prefill_gpu(q, pb.cu_q, pb.ctx_before, pb.block_table)
    again, lse2 = layer.prefill_gpu(q, pb.cu_q, pb.ctx_before, pb.block_table)
    assert torch.equal(again, out) and torch.equal(lse2, lse), "a second call differs"
    rows = np.sort(wl.rng_for(92).choice(pb.T, size=min(pb.T, 400), replace=False)).astype(np.int64)
    seq = np.searchsorted(pb.cu_q, rows, side="right") - 1
    start = np.searchsorted(seq, np.arange(pb.B + 1), side="left").astype(np.int32)
    pos = pb.ctx_before[seq] + (rows - pb.cu_q[seq])
    ref, ref_lse = orc.attn_rows(layer.shape, wl.to_bits(q), layer.okc, layer.ovc, pb.block_table, start, rows.astype(np.int32), pos.astype(np.int32))
    compare("prefill", out, ref, "bf16", rows=rows)
    compare_lse("prefill", lse, ref_lse, "bf16", rows=rows, bf16_row_sum=True)
    # several layers that share one plan: the merge counters are as the first left them
    layer.ctx.set_option(binding.OPT_PREFILL_REUSE_PLAN, 1)
    cu, cb, bt, qd = dev_i32(pb.cu_q), dev_i32(pb.ctx_before), dev_i32(pb.block_table), q.cuda()
    for i in range(3):
        o = torch.full_like(out, float("nan"))
        layer.ctx.attn_prefill(qd, layer.kc, layer.vc, cu, cb, bt, o, None, max_q_len=int(new.max()))
        assert torch.equal(o, out), f"layer {i} with the shared plan differs"
    layer.close()


def test_keys_of_minus_infinity_at_the_beginning_of_pieces():
    """Keys whose scores are minus infinity weigh nothing, also where they fill whole key steps and a piece begins there."""
    Hq, Hkv, cached, new = 40, 8, 4000, 8
    model = wl.ModelShape("shares", Hq, Hkv, 128, 1, "bf16")
    say("prefill, keys of minus infinity in whole key steps")
    pb = wl.prefill_batch(model, np.asarray([new], dtype=np.int32), 93, ctx_before=np.asarray([cached], dtype=np.int32))
    layer = Layer(model, pb.num_blocks, 1, pb.block_table.shape[1], oracle_cache=False)
    n = cached + new
    k = torch.zeros((n, Hkv, 128), dtype=torch.bfloat16)
    k[300:3700, :, 0] = -float("inf")
    v = wl.randn((n, Hkv, 128), "bf16", 6)
    layer.ctx.kv_append(layer.kc, layer.vc, k.cuda(), v.cuda(), dev_i32([0, n]), dev_i32([0]), dev_i32(pb.block_table))
    q = torch.zeros((new, Hq, 128), dtype=torch.bfloat16)
    q[:, :, 0] = 1.0
    out, lse = layer.prefill_gpu(q, pb.cu_q, pb.ctx_before, pb.block_table)
    # equal weights on all other keys: running means of V
    seen = torch.cat([torch.arange(300), torch.arange(3700, n)])
    for i in range(new):
        keys = seen[seen <= cached + i]
        ref = v[keys].double().mean(0).repeat_interleave(Hq // Hkv, dim=0)
        assert (out[i].double().cpu() - ref).abs().max() <= 1e-2
        assert (lse[i].double().cpu() - np.log(len(keys))).abs().max() <= 1e-3
    layer.close()
