"""The matrix-core kernels for every layout but (bf16, head size 128) against the fp64 CPU oracle: head sizes at and
beside the edges of a matrix step (16 elements of fp32, 32 of bf16), every group shape of the 16 columns, contexts at
the edges of blocks, wavefront rounds and slices, with and without a cached prefix."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2504_18154_amd import workloads as wl
from tests.parity_util import Layer, compare, compare_lse, dev_i32, say

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 4, 2, 1), ("f32", 20, 4, 2), ("f32", 64, 4, 2), ("f32", 100, 3, 3), ("f32", 128, 6, 3), ("f32", 160, 16, 1),
          ("f32", 256, 5, 1), ("bf16", 8, 2, 2), ("bf16", 40, 10, 2), ("bf16", 64, 32, 8), ("bf16", 72, 7, 1), ("bf16", 80, 8, 8),
          ("bf16", 96, 8, 2), ("bf16", 120, 16, 1), ("bf16", 136, 4, 2), ("bf16", 192, 3, 1), ("bf16", 256, 8, 1)]


@pytest.mark.parametrize("dtype,D,Hq,Hkv", SHAPES, ids=[f"{s[0]}-d{s[1]}-{s[2]}x{s[3]}" for s in SHAPES])
def test_prefill_and_decode_against_the_oracle(dtype, D, Hq, Hkv):
    """One prefill batch (an empty prompt, one token, block edges, several tiles; some behind a cached prefix), then
    two decode steps, the second with the append fused in, then forced slices of the context."""
    from paper_2504_18154_amd import binding
    model = wl.ModelShape(f"{dtype}-d{D}", Hq, Hkv, D, 1, dtype)
    before = np.array([0, 0, 5, 0, 16, 300, 0, 31, 0], dtype=np.int32)
    new = np.array([1, 0, 1, 15, 17, 40, 64, 33, 150], dtype=np.int32)
    say(f"{dtype}, head size {D}, heads {Hq}/{Hkv}: prefill {new.tolist()} behind {before.tolist()}")
    pb = wl.prefill_batch(model, before + new, 300 + D, grow=3)
    B = len(new)
    layer = Layer(model, pb.num_blocks, B, pb.block_table.shape[1])
    zero = np.zeros(B, dtype=np.int32)
    rows = lambda n, h, seed: wl.randn((int(n), h, D), dtype, seed)
    layer.append(rows(before.sum(), Hkv, 1), rows(before.sum(), Hkv, 2), wl.cu_from_lengths(before), zero, pb.block_table)
    cu = wl.cu_from_lengths(new)
    layer.append(rows(new.sum(), Hkv, 3), rows(new.sum(), Hkv, 4), cu, before, pb.block_table)
    q = rows(new.sum(), Hq, 5)
    out, lse = layer.prefill_gpu(q, cu, before, pb.block_table)
    ref, ref_lse = layer.prefill_oracle(q, cu, before, pb.block_table)
    compare("prefill", out, ref, dtype)
    compare_lse("prefill", lse, ref_lse, dtype)

    live = np.flatnonzero(before + new > 0)          # (the empty sequence has no context to decode over)
    table, ctx = pb.block_table[live], (before + new)[live]
    B = len(live)
    ones = wl.cu_from_lengths([1] * B)
    for step in range(2):
        q, k, v = rows(B, Hq, 10 + step), rows(B, Hkv, 20 + step), rows(B, Hkv, 30 + step)
        if step == 0:
            layer.append(k, v, ones, ctx, table, max_new_len=1)
            out, lse = layer.decode_gpu(q, table, ctx + 1)
        else:
            orc.kv_append(layer.shape, layer.okc, layer.ovc, wl.to_bits(k), wl.to_bits(v), ones, ctx, table)
            out = torch.full((B, Hq, D), float("nan"), dtype=q.dtype, device="cuda")
            lse = torch.full((B, Hq), float("nan"), dtype=torch.float32, device="cuda")
            layer.ctx.attn_decode_append(q.cuda(), k.cuda(), v.cuda(), layer.kc, layer.vc, dev_i32(table), dev_i32(ctx + 1), out,
                                         int(ctx.max()) + 1, lse)
        ctx = ctx + 1
        layer.assert_cache_bit_exact()
        ref, ref_lse = layer.decode_oracle(q, table, ctx)
        compare(f"decode step {step}", out, ref, dtype)
        compare_lse(f"decode step {step}", lse, ref_lse, dtype)
    for split in (64, 192):
        layer.ctx.set_option(binding.OPT_DECODE_SPLIT_TOKENS, split)
        out, lse = layer.decode_gpu(q, table, ctx)
        compare(f"decode in slices of {split}", out, ref, dtype)
        compare_lse(f"decode in slices of {split}", lse, ref_lse, dtype)
    layer.close()


@pytest.mark.parametrize("dtype,D,heads", [("bf16", 24, (9, 1)), ("bf16", 32, (32, 2)), ("bf16", 64, (8, 1)), ("f32", 36, (15, 1)), ("bf16", 88, (32, 2)), ("f32", 128, (16, 1)), ("bf16", 104, (4, 4)),
                                           ("bf16", 128, (16, 1))], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_decode_of_whole_contexts_with_one_row_to_a_wavefront_or_two(dtype, D, heads):
    """Groups of up to 16 rows over eight wavefronts, contexts that end in the first block, in some of the wavefronts' and in all; then an infinite V element, which takes the rows of its
    sequence and K/V head to the other way through the kernel's end."""
    from paper_2504_18154_amd import binding
    model = wl.ModelShape(f"{dtype}-d{D}", *heads, D, 1, dtype)
    lens = np.asarray([1, 16, 17, 70, 128, 129, 9, 400, 33], dtype=np.int32)
    say(f"{dtype}, head size {D}, heads {heads}: decode of whole contexts")
    pb = wl.prefill_batch(model, lens, 83)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v, q = (wl.randn((n, h, D), dtype, s) for s, n, h in ((1, pb.T, heads[1]), (2, pb.T, heads[1]), (3, pb.B, heads[0])))
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
    out, lse = layer.decode_gpu(q, pb.block_table, lens)
    compare("decode", out, ref, dtype)
    compare_lse("decode", lse, ref_lse, dtype)
    v[int(pb.cu_q[3]) + 40, 0, 5] = float("inf")   # of the fourth sequence
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    got, glse = layer.decode_gpu(q, pb.block_table, lens)
    layer.ctx.set_option(binding.OPT_FORCE_PLAIN, 1)
    want, _ = layer.decode_gpu(q, pb.block_table, lens)
    G, fin = heads[0] // heads[1], torch.isfinite(want)
    assert torch.isinf(want[3, :G, 5].float()).all() and int((~fin).sum()) == G
    assert torch.equal(torch.isfinite(got), fin) and torch.equal(torch.isinf(got), torch.isinf(want))
    compare_lse("decode, an infinite value", glse, ref_lse, dtype)
    others = [b for b in range(pb.B) if b != 3]
    assert torch.equal(got[others], out[others]) and torch.equal(glse[others], lse[others])
    layer.close()


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("bf16", 64)])
def test_decode_over_contexts_of_several_slices(dtype, D):
    """Contexts above 1024 tokens are cut into slices whose states are merged, the newest token in the last one:
    lengths around the slices' edges, alone (slices of 256) and beside many sequences (slices of 1024)."""
    model = wl.ModelShape(f"{dtype}-d{D}", 4, 2, D, 1, dtype)
    for lens in ([2049], [1024, 1025, 1, 2047, 2048] + [40] * 130):
        lens = np.asarray(lens, dtype=np.int32)
        say(f"{dtype}, head size {D}: decode over up to {lens.max()} tokens, {len(lens)} sequences")
        pb = wl.prefill_batch(model, lens, 77)
        layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
        k, v = (wl.randn((pb.T, 2, D), dtype, s) for s in (1, 2))
        layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
        q = wl.randn((pb.B, 4, D), dtype, 3)
        ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
        out, lse = layer.decode_gpu(q, pb.block_table, lens)
        compare("decode", out, ref, dtype)
        compare_lse("decode", lse, ref_lse, dtype)
        last = torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)
        fused, fused_lse = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
        layer.wipe_newest(pb.block_table, lens)
        layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens),
                                     fused, int(lens.max()), fused_lse)
        torch.cuda.synchronize()
        assert torch.equal(fused, out) and torch.equal(fused_lse, lse), "the fused append changes the result"
        layer.assert_cache_bit_exact()
        layer.close()


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("bf16", 96)])
def test_infinite_values_reach_only_the_rows_that_see_them(dtype, D):
    """An infinite V element: rows before it must not notice (its weight there is a zero that must not meet it), rows
    that see it are infinite in that element and finite in the others, as in the plain kernels."""
    from paper_2504_18154_amd import binding
    model = wl.ModelShape(f"{dtype}-d{D}", 4, 2, D, 1, dtype)
    pb = wl.prefill_batch(model, [70, 20], 78)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v, q = (wl.randn((pb.T, h, D), dtype, s) for s, h in ((1, 2), (2, 2), (3, 4)))
    v[33, 1, 5] = float("inf")
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    got, glse = layer.prefill_gpu(q, pb.cu_q, pb.ctx_before, pb.block_table)
    qd = q[torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)]
    gd, _ = layer.decode_gpu(qd, pb.block_table, pb.q_len)
    layer.ctx.set_option(binding.OPT_FORCE_PLAIN, 1)
    want, wlse = layer.prefill_gpu(q, pb.cu_q, pb.ctx_before, pb.block_table)
    wd, _ = layer.decode_gpu(qd, pb.block_table, pb.q_len)
    assert torch.equal(torch.isfinite(got), torch.isfinite(want)) and torch.equal(torch.isfinite(gd), torch.isfinite(wd))
    assert torch.isfinite(got[:33]).all() and torch.isinf(got[33:70, 2:, 5]).all() and torch.isinf(gd[0, 2:, 5]).all()
    # both kernels are within half a spacing of the same sums: a spacing of bf16 (2^-7 of |o| < 4) apart at most, fp32 by its sums
    tol = 2.0 ** -6 if dtype == "bf16" else 1e-5
    fin = torch.isfinite(want)
    assert (got[fin].float() - want[fin].float()).abs().max() <= tol
    assert (gd.float() - wd.float())[torch.isfinite(wd)].abs().max() <= tol
    assert (glse - wlse).abs().max() <= 1e-4
    layer.close()


@pytest.mark.parametrize("dtype,D,prompts", [("f32", 64, 1), ("bf16", 96, 1), ("f32", 64, 12), ("bf16", 96, 12)],
                         ids=["f32-d64", "bf16-d96", "f32-d64-shared-rows", "bf16-d96-shared-rows"])
def test_infinite_values_in_long_contexts_and_shared_rows(dtype, D, prompts):
    """The same where the row that is taken again is one of a tile whose rows are shared out (12 prompts with 32 query heads), and
    where a decode step's context is cut into slices: infinities in the first, a middle and the last of nine, the last one in
    the token that the fused append brings."""
    from paper_2504_18154_amd import binding
    model = wl.ModelShape(f"{dtype}-d{D}", 32, 2, D, 1, dtype)
    lens = np.asarray([2300] if prompts == 1 else [70] * prompts, dtype=np.int32)
    pb = wl.prefill_batch(model, lens, 79)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v, q = (wl.randn((pb.T, h, D), dtype, s) for s, h in ((1, 2), (2, 2), (3, 32)))
    bad = [(33, 5), (1100, 6), (2299, 7)] if prompts == 1 else [(33, 5), (150, 6), (pb.T - 1, 7)]
    for t, d in bad:
        v[t, 1, d] = float("inf")
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    last = torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)
    rows = slice(None) if prompts > 1 else slice(1000, 1200)  # (the plain kernels' time; a chunk behind 1000 cached tokens)
    cu, before = (pb.cu_q, pb.ctx_before) if prompts > 1 else (wl.cu_from_lengths([200]), np.asarray([1000], np.int32))

    def both():
        out, lse = layer.prefill_gpu(q[rows], cu, before, pb.block_table)
        layer.wipe_newest(pb.block_table, lens)
        dec = torch.full((pb.B, 32, D), float("nan"), dtype=q.dtype, device="cuda")
        dec_lse = torch.full((pb.B, 32), float("nan"), dtype=torch.float32, device="cuda")
        layer.ctx.attn_decode_append(q[last].cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens),
                                     dec, int(lens.max()), dec_lse)
        torch.cuda.synchronize()
        return out, lse, dec, dec_lse

    got = both()
    layer.assert_cache_bit_exact()
    layer.ctx.set_option(binding.OPT_FORCE_PLAIN, 1)
    want = both()
    tol = 2.0 ** -6 if dtype == "bf16" else 1e-5  # (as above)
    for g, w in zip(got[::2], want[::2]):
        fin = torch.isfinite(w)
        assert torch.equal(torch.isfinite(g), fin) and torch.equal(torch.isinf(g), torch.isinf(w))
        assert not fin.all() and (g[fin].float() - w[fin].float()).abs().max() <= tol
    for g, w in zip(got[1::2], want[1::2]):
        assert (g - w).abs().max() <= 1e-4
    layer.close()


@pytest.mark.parametrize("dtype,D,Hq,Hkv,before,new", [
    ("f32", 64, 32, 2, [1021, 1023, 1024, 2100, 0, 3, 60] + [5] * 6, [3] * 13), ("bf16", 96, 32, 2, [1021, 1023, 1024, 2100] + [0] * 9, [3] * 13),
    ("f32", 256, 32, 2, [1022, 1030] + [0] * 10, [2, 5] + [1] * 10), ("f32", 64, 4, 2, [4090, 8300], [7, 3]), ("bf16", 80, 4, 4, [4094, 60], [4, 9])],
    ids=["f32-d64-shared-rows", "bf16-d96-shared-rows", "f32-d256-shared-rows", "f32-d64-shared-keys", "bf16-d80-shared-keys"])
def test_prefill_behind_long_prefixes(dtype, D, Hq, Hkv, before, new):
    """A wavefront walks its blocks 64 ids at a time: rows that see more than 1024 keys (rows shared out: each wavefront walks them
    all), or more than 4096 (keys shared out: every fourth block), at and beside the first change of ids, and the second."""
    model = wl.ModelShape(f"{dtype}-d{D}", Hq, Hkv, D, 1, dtype)
    before, new = np.asarray(before, np.int32), np.asarray(new, np.int32)
    say(f"{dtype}, head size {D}, heads {Hq}/{Hkv}: prefill {new.tolist()} behind {before.tolist()}")
    pb = wl.prefill_batch(model, before + new, 92)
    layer = Layer(model, pb.num_blocks, len(new), pb.block_table.shape[1])
    rows = lambda n, h, seed: wl.randn((int(n), h, D), dtype, seed)
    layer.append(rows(before.sum(), Hkv, 1), rows(before.sum(), Hkv, 2), wl.cu_from_lengths(before), np.zeros_like(before), pb.block_table)
    cu = wl.cu_from_lengths(new)
    layer.append(rows(new.sum(), Hkv, 3), rows(new.sum(), Hkv, 4), cu, before, pb.block_table)
    q = rows(new.sum(), Hq, 5)
    out, lse = layer.prefill_gpu(q, cu, before, pb.block_table)
    ref, ref_lse = layer.prefill_oracle(q, cu, before, pb.block_table)
    compare("prefill", out, ref, dtype)
    compare_lse("prefill", lse, ref_lse, dtype)
    layer.close()


@pytest.mark.parametrize("dtype,D,Hq,Hkv", [("f32", 64, 16, 2), ("bf16", 64, 32, 8), ("bf16", 80, 24, 8), ("bf16", 256, 8, 1), ("f32", 160, 8, 4)],
                         ids=["f32-d64", "bf16-d64", "bf16-d80", "bf16-d256", "f32-d160"])
def test_prefill_of_many_short_prompts(dtype, D, Hq, Hkv):
    """Batches that share out the rows of a tile instead of its keys (many short prompts), some behind cached tokens: more
    sequences than one round of the search for a tile's sequence holds, lengths around the tiles' edges, empty ones."""
    model = wl.ModelShape(f"{dtype}-d{D}", Hq, Hkv, D, 1, dtype)
    rng = np.random.default_rng(D)
    new = np.r_[0, 0, 1, 16, 17, 63, 64, 65, 0, 130, rng.integers(0, 50, size=80)].astype(np.int32)
    before = np.where(rng.random(len(new)) < 0.3, rng.integers(0, 90, size=len(new)), 0).astype(np.int32)
    say(f"{dtype}, head size {D}: {len(new)} prompts, {new.sum()} tokens")
    pb = wl.prefill_batch(model, np.maximum(before + new, 1), 91)
    layer = Layer(model, pb.num_blocks, len(new), pb.block_table.shape[1])
    rows = lambda n, h, seed: wl.randn((int(n), h, D), dtype, seed)
    layer.append(rows(before.sum(), Hkv, 1), rows(before.sum(), Hkv, 2), wl.cu_from_lengths(before), np.zeros_like(before), pb.block_table)
    cu = wl.cu_from_lengths(new)
    layer.append(rows(new.sum(), Hkv, 3), rows(new.sum(), Hkv, 4), cu, before, pb.block_table)
    layer.assert_cache_bit_exact()
    q = rows(new.sum(), Hq, 5)
    out, lse = layer.prefill_gpu(q, cu, before, pb.block_table)
    ref, ref_lse = layer.prefill_oracle(q, cu, before, pb.block_table)
    compare("prefill", out, ref, dtype)
    compare_lse("prefill", lse, ref_lse, dtype)
    layer.close()


def test_workspace_does_not_hold_a_tile_list_for_layouts_that_have_none():
    """The list of query tiles is what the workspace grows by with the pool: G records of 80 bytes per 128 tokens for (bf16,
    128), and nothing for the other layouts, whatever their group size."""
    from paper_2504_18154_amd import binding
    blocks = 1 << 16
    for dtype, D, Hq, want in (("f32", 64, 32, 0), ("bf16", 64, 2, 0), ("bf16", 128, 2, 80 * blocks // 8), ("bf16", 128, 32, 16 * 80 * blocks // 8)):
        sizes = []
        for n in (8, 8 + blocks):
            ctx = binding.Context(Hq, 2, D, n, dtype, 1, 8)
            sizes.append(ctx.workspace_bytes())
            ctx.close()
        assert sizes[1] - sizes[0] == want, (dtype, D, Hq, sizes)
