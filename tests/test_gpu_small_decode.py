"""Decode of small (bf16, head size 128) batches, which run in one launch: at the edges of the rule that picks that
kernel, of its slices and of its wavefronts' rounds, against the fp64 CPU oracle, called twice (the second call finds
the merge counters as the first one left them) and with the append fused in."""
import numpy as np
import pytest
import torch

from paper_2504_18154_amd import binding
from paper_2504_18154_amd import workloads as wl
from tests.parity_util import Layer, compare, compare_lse, dev_i32, say

pytestmark = pytest.mark.gpu

CASES = [((40, 8), [1]), ((40, 8), [16, 17, 127, 128, 129]), ((40, 8), [1024]), ((64, 8), [1025]), ((5, 1), [4097, 255, 257, 1, 513]),
         ((8, 1), [9000]), ((16, 1), [1023] * 3 + [2048] * 20), ((40, 8), [30] * 31 + [1024]),          # 256 (sequence, K/V head)s
         ((40, 8), [30] * 32 + [512]),                                                                  # 264: four wavefronts each
         ((64, 8), [17] * 60 + [1, 496, 511, 512]), ((52, 52), [100] * 9), ((3, 3), [700, 2000, 40])]


@pytest.mark.parametrize("heads,lens", CASES, ids=[f"{h[0]}x{h[1]}-B{len(n)}-L{max(n)}" for h, n in CASES])
def test_small_decode_batches(heads, lens):
    model = wl.ModelShape("small", heads[0], heads[1], 128, 1, "bf16")
    lens = np.asarray(lens, dtype=np.int32)
    say(f"decode, heads {heads}, {len(lens)} sequences up to {lens.max()} tokens")
    pb = wl.prefill_batch(model, lens, 55)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v = (wl.randn((pb.T, model.Hkv, 128), "bf16", s) for s in (1, 2))
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, model.Hq, 128), "bf16", 3)
    ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
    out, lse = layer.decode_gpu(q, pb.block_table, lens)
    compare("decode", out, ref, "bf16")
    compare_lse("decode", lse, ref_lse, "bf16")
    again, lse2 = layer.decode_gpu(q, pb.block_table, lens)
    assert torch.equal(again, out) and torch.equal(lse2, lse), "a second call differs"
    last = torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)
    fused = torch.full_like(out, float("nan"))
    layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens),
                                 fused, int(lens.max()))
    no = torch.full_like(out, float("nan"))
    st = binding.attn_decode_noalloc(layer.ctx.layout, q.cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), no, int(lens.max()))
    assert st == binding.OK
    torch.cuda.synchronize()
    assert torch.equal(fused, out), "the fused append changes the result"
    assert torch.equal(no, out), "the call without a context differs"
    layer.assert_cache_bit_exact()
    layer.close()
