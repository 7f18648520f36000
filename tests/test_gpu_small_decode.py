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

# In slices of the small-batch kernel, most of them one each (test_decode_slices.py asserts it):
CASES = [((40, 8), [1, 513]), ((40, 8), [16, 17, 127, 128, 129, 385]), ((40, 8), [1024]), ((64, 8), [1025]), ((5, 1), [4097, 255, 257, 1, 513]),
         ((8, 1), [9000]), ((16, 1), [1023] * 3 + [2048] * 20), ((40, 8), [30] * 31 + [1024]),          # 256 (sequence, K/V head)s
         ((64, 8), [17] * 28 + [1, 496, 511, 512]), ((52, 52), [100, 100, 100, 400]), ((3, 3), [700, 2000, 40])]
# decoded whole:
WHOLE = [((40, 8), [1]), ((40, 8), [16, 17, 127, 128, 129]), ((40, 8), [30] * 32 + [512]), ((64, 8), [17] * 60 + [1, 496, 511, 512]), ((52, 52), [100] * 9)]


@pytest.mark.parametrize("heads,lens", CASES + WHOLE, ids=[f"{h[0]}x{h[1]}-B{len(n)}-L{max(n)}" for h, n in CASES + WHOLE])
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
    fused, fused_lse = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
    layer.wipe_newest(pb.block_table, lens)
    layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens),
                                 fused, int(lens.max()), fused_lse)
    no = torch.full_like(out, float("nan"))
    st = binding.attn_decode_noalloc(layer.ctx.layout, q.cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), no, int(lens.max()))
    assert st == binding.OK
    torch.cuda.synchronize()
    assert torch.equal(fused, out) and torch.equal(fused_lse, lse), "the fused append changes the result"
    assert torch.equal(no, out), "the call without a context differs"
    layer.assert_cache_bit_exact()
    layer.close()


@pytest.mark.parametrize("lens,bound", [([9000, 20], 600), ([9000, 20], 16), ([30] * 32 + [4200], 512)], ids=["eight-wavefronts", "whole-by-one", "four-wavefronts"])
def test_a_bound_on_the_lengths_that_is_too_low_costs_time_only(lens, bound):
    """max_ctx_len is to be an upper bound; the persistent kernel never used it, and where this kernel's grid ends short of a
    context its last slice takes the rest: more blocks than the 64 ids a wavefront holds, so it walks them in windows, as does the
    kernel for whole contexts."""
    model = wl.ModelShape("small", 40, 8, 128, 1, "bf16")
    lens = np.asarray(lens, dtype=np.int32)
    pb = wl.prefill_batch(model, lens, 56)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    layer.append(*(wl.randn((pb.T, 8, 128), "bf16", s) for s in (1, 2)), pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, 40, 128), "bf16", 3)
    ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
    out, lse = layer.decode_gpu(q, pb.block_table, lens, max_ctx_len=bound)
    compare("decode", out, ref, "bf16")
    compare_lse("decode", lse, ref_lse, "bf16")
    layer.close()


@pytest.mark.parametrize("lens", [[300, 40], [700, 40], [3000, 40]], ids=["whole", "one-slice", "slices"])
def test_infinite_values_reach_only_their_own_elements(lens):
    """Infinite V elements (the weights' remainders are zero for some keys, and must not make them NaN), one of them in the token
    that the fused append brings: infinite there, elsewhere as the plain kernels have it."""
    model = wl.ModelShape("small", 40, 8, 128, 1, "bf16")
    lens = np.asarray(lens, dtype=np.int32)
    pb = wl.prefill_batch(model, lens, 57)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v = (wl.randn((pb.T, 8, 128), "bf16", s) for s in (1, 2))
    for t, g, d in ((33, 1, 5), (int(lens[0]) // 2, 1, 6), (int(lens[0]) - 1, 2, 7)):
        v[t, g, d] = float("inf")
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, 40, 128), "bf16", 3)
    last = torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)
    res = []
    for plain in (0, 1):
        layer.ctx.set_option(binding.OPT_FORCE_PLAIN, plain)
        layer.wipe_newest(pb.block_table, lens)
        out = torch.full((pb.B, 40, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), out,
                                     int(lens.max()))
        torch.cuda.synchronize()
        layer.assert_cache_bit_exact()
        res.append(out.float())
    got, want = res
    fin = torch.isfinite(want)
    assert torch.isinf(want[0, 5:10, 5:7]).all() and torch.isinf(want[0, 10:15, 7]).all() and int((~fin).sum()) == 15
    assert torch.equal(torch.isfinite(got), fin) and torch.equal(torch.isinf(got), torch.isinf(want))
    assert (got[fin] - want[fin]).abs().max() <= 2.0 ** -6   # half a spacing of bf16 (2^-7 of |o| < 4) each, and the weights' 2^-17
    layer.close()


@pytest.mark.parametrize("each", [15, 19], ids=["B40", "B48"])
def test_sequences_without_tokens_are_passed_over(each):
    """Lengths of zero first, in the middle, several in a row, and last, among up to 1500 tokens; with a context and without.  48 sequences
    (384 (sequence, K/V head)s for 256 workgroups) are cut on the device, 40 take balanced slices, two workgroups per CU
    (test_decode_slices.py asserts it; the persistent kernel's empty sequences are in test_gpu_decode_sliced.py)."""
    model = wl.ModelShape("30B-heads", 40, 8, 128, 1, "bf16")
    rng = np.random.default_rng(58)
    lens = np.r_[0, 0, 700, 0, rng.integers(1, 600, size=each), 0, 0, 1500, 0, rng.integers(1, 600, size=each), 16, 0].astype(np.int32)
    pb = wl.prefill_batch(model, np.maximum(lens, 1), 59)
    layer = Layer(model, pb.num_blocks, len(lens), pb.block_table.shape[1])
    layer.append(*(wl.randn((int(lens.sum()), 8, 128), "bf16", s) for s in (1, 2)), wl.cu_from_lengths(lens), np.zeros_like(lens), pb.block_table)
    q = wl.randn((len(lens), 40, 128), "bf16", 3)
    live = np.flatnonzero(lens > 0)
    ref, ref_lse = layer.decode_oracle(q[live], pb.block_table[live], lens[live])
    out, lse = layer.decode_gpu(q, pb.block_table, lens)
    no = torch.full_like(out, float("nan"))
    assert binding.attn_decode_noalloc(layer.ctx.layout, q.cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), no, 1500) == binding.OK
    torch.cuda.synchronize()
    compare("rows of the non-empty sequences", out, ref, "bf16", rows=live)
    compare_lse("rows of the non-empty sequences", lse, ref_lse, "bf16", rows=live)
    compare("without a context", no, ref, "bf16", rows=live)
    layer.close()


# Several sequences of very different lengths: at the edges of blocks, of the wavefronts' rounds and of the rule that leaves contexts
# whole; empty sequences; as many sequences as a wavefront has lanes.  Which of them are cut into balanced slices with the caller's bound
# at the longest and 3000 tokens above it: PATHS in test_decode_slices.py.
RAGGED = [((40, 8), [769, 1]), ((40, 8), [2000, 128, 129, 127, 16, 17, 0, 1024]), ((64, 8), [1025] * 20), ((5, 1), [0, 3000, 0, 0, 2999, 1, 0]),
          ((16, 1), [4095, 4096, 4097] + [1] * 61), ((3, 3), [900, 700, 5000]), ((52, 52), [800, 1500]), ((8, 1), [30000, 20, 700]),
          ((40, 8), [600] * 36 + [0, 1, 128, 1000]), ((16, 4), [1 + 17 * i for i in range(64)])]
# Balanced slices on one workgroup per CU (8 wavefronts) or two (4), with what the bound may lie above the longest context: empty
# sequences first, last and in a row; one long context beside many tiny ones; several trials until the slices fit.
BALANCED = [((40, 8), [0, 0, 3000, 0, 0, 0, 40, 0, 2999, 1, 0, 0], 3000, 8), ((8, 1), [12000] + [20] * 40, 3000, 8), ((40, 8), [2000] * 20, 3000, 8),
            ((5, 1), [0] * 20 + [3000, 0, 0, 2999, 1, 0] + [5] * 30, 3000, 8), ((40, 8), [4000 - 7 * i for i in range(20)], 900, 8), ((16, 4), [0] * 39 + [2500], 2000, 8),
            ((40, 8), [0, 0, 0, 1100, 0] + [300] * 18 + [0], 1500, 4), ((40, 8), [1100, 1099] + [1030] * 36 + [1, 0], 700, 4),
            ((16, 4), [1200] + [20] * 62 + [0], 1100, 4), ((52, 52), [0, 2500, 20, 1025], 300, 4), ((8, 1), [290000], 300000, 4)]


@pytest.mark.parametrize("heads,lens", RAGGED, ids=[f"{h[0]}x{h[1]}-B{len(n)}-L{max(n)}" for h, n in RAGGED])
@pytest.mark.parametrize("loose", [False, True], ids=["tight", "loose"])
def test_ragged_lengths(heads, lens, loose):
    _against_the_oracle(heads, lens, max(lens) + (3000 if loose else 0))


@pytest.mark.parametrize("heads,lens,above,waves", BALANCED, ids=[f"{c[0][0]}x{c[0][1]}-B{len(c[1])}-L{max(c[1])}" for c in BALANCED])
@pytest.mark.parametrize("loose", [False, True], ids=["tight", "loose"])
def test_balanced_slices(heads, lens, above, waves, loose):
    _against_the_oracle(heads, lens, max(lens) + (above if loose else 0))


def _against_the_oracle(heads, lens, bound):
    model = wl.ModelShape("balanced", heads[0], heads[1], 128, 1, "bf16")
    lens = np.asarray(lens, dtype=np.int32)
    say(f"decode, heads {heads}, lengths {lens.tolist()}, the caller's bound {bound}")
    pb = wl.prefill_batch(model, lens, 57)
    table = np.pad(pb.block_table, ((0, 0), (0, (bound + 15) // 16 - pb.block_table.shape[1])), constant_values=2**30)  # never read there
    layer = Layer(model, pb.num_blocks, pb.B, table.shape[1])
    k, v = (wl.randn((pb.T, model.Hkv, 128), "bf16", s) for s in (1, 2))
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, model.Hq, 128), "bf16", 3)
    some = np.flatnonzero(lens)
    ref, ref_lse = layer.decode_oracle(q[torch.as_tensor(some)], pb.block_table[some], lens[some])
    out, lse = layer.decode_gpu(q, table, lens, bound)
    idx = torch.as_tensor(some, device="cuda")
    compare("decode", out[idx], ref, "bf16")
    compare_lse("decode", lse[idx], ref_lse, "bf16")
    last = torch.as_tensor(np.maximum(pb.cu_q[1:] - 1, 0), dtype=torch.long)
    layer.wipe_newest(pb.block_table[some], lens[some])
    bt, tot = dev_i32(table), dev_i32(lens)
    for call in range(3):
        fused, fused_lse = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
        layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, bt, tot, fused, bound, fused_lse)
        assert torch.equal(fused[idx], out[idx]) and torch.equal(fused_lse[idx], lse[idx]), f"call {call} with the append fused in differs"
    no = torch.full_like(out, float("nan"))
    assert binding.attn_decode_noalloc(layer.ctx.layout, q.cuda(), layer.kc, layer.vc, bt, tot, no, bound) == binding.OK
    torch.cuda.synchronize()
    assert torch.equal(no[idx], out[idx]), "the call without a context differs"
    layer.assert_cache_bit_exact()
    layer.close()


@pytest.mark.parametrize("dtype,heads,D,lens", [("f32", (4, 2), 64, [700, 337, 128, 129, 1]), ("f32", (6, 3), 128, [400, 225, 16]), ("f32", (4, 2), 256, [200, 65, 64, 63]),
                                                ("bf16", (16, 2), 192, [700, 512]), ("bf16", (8, 1), 256, [800, 400, 17]), ("bf16", (8, 2), 96, [1024, 1023])],
                         ids=lambda x: str(x).replace(" ", ""))
def test_short_slices_of_other_layouts(dtype, heads, D, lens):
    """Contexts that other layouts cut below 1024 tokens: against the oracle, and with the append fused in, three times."""
    model = wl.ModelShape("other", heads[0], heads[1], D, 1, dtype)
    lens = np.asarray(lens, dtype=np.int32)
    say(f"decode, {dtype}, head size {D}, heads {heads}, lengths {lens.tolist()}")
    pb = wl.prefill_batch(model, lens, 60)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v = (wl.randn((pb.T, model.Hkv, D), dtype, s) for s in (1, 2))
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, model.Hq, D), dtype, 3)
    ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
    out, lse = layer.decode_gpu(q, pb.block_table, lens)
    compare("decode", out, ref, dtype)
    compare_lse("decode", lse, ref_lse, dtype)
    last = torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)
    layer.wipe_newest(pb.block_table, lens)
    for call in range(3):
        fused = torch.full_like(out, float("nan"))
        layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), fused, int(lens.max()))
        torch.cuda.synchronize()
        assert torch.equal(fused, out), f"call {call} with the append fused in differs"
    layer.assert_cache_bit_exact()
    layer.close()
