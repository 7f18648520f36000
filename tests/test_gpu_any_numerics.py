"""What the kernels of attn_any_mfma.hip owe at the edges of fp32, each case with a closed form or an fp64 sum beside it; the
plain kernels (ECOSERVE_OPT_FORCE_PLAIN) are held to the same."""
import math

import numpy as np
import pytest
import torch

from paper_2504_18154_amd import binding
from paper_2504_18154_amd import workloads as wl
from tests.parity_util import dev_i32, say

pytestmark = pytest.mark.gpu

# (type, head size, K/V heads): fp32, bf16, and the layout whose small decode batches take the same kernel (with weights of
# 16 bits and none below 2^-126, where its other kernels have 8 bits) or the one for whole contexts beside it
LAYOUTS = [("f32", 64, 2), ("bf16", 64, 2), ("bf16", 128, 2)]
IDS = ["f32-d64", "bf16-d64", "bf16-d128"]


class Scored:
    """B equal sequences whose key t scores log2_w[t] in log2 units for every query: the softmax scale is ln 2 (which times
    log2 e is 1 in fp32), queries are the first unit vector and key t's first element is log2_w[t].  values: [n, D]."""

    def __init__(self, dtype, D, Hkv, log2_w, values, B=1, before=None):
        n = len(log2_w)
        self.B, self.n, self.D, self.Hq, self.Hkv, self.dtype = B, n, D, 2 * Hkv, Hkv, dtype
        table, num_blocks = wl.make_block_table(wl.rng_for(5), np.full(B, n))
        table = np.pad(table, ((0, 0), (0, max(0, 64 - table.shape[1]))), constant_values=-1)   # (room for a bound above the lengths)
        self.ctx = binding.Context(self.Hq, Hkv, D, num_blocks, dtype, B, table.shape[1], softmax_scale=math.log(2.0))
        self.kc, self.vc = self.ctx.new_cache()
        dt = self.ctx.torch_dtype
        k = torch.zeros((n, Hkv, D), dtype=torch.float64)
        k[:, :, 0] = torch.as_tensor(np.asarray(log2_w, dtype=np.float64))[:, None]
        v = torch.as_tensor(np.asarray(values, dtype=np.float64))[:, None, :].expand(n, Hkv, D)
        assert torch.equal(k.to(dt).double(), k) and torch.equal(v.to(dt).double(), v), "inputs have to be exact in the storage type"
        self.table, zero = dev_i32(table), dev_i32(np.zeros(B))
        self.lens, self.before = dev_i32(np.full(B, n)), dev_i32(np.full(B, before or 0))
        self.new = n - (before or 0)
        self.ctx.kv_append(self.kc, self.vc, k.to(dt).repeat(B, 1, 1).cuda(), v.to(dt).repeat(B, 1, 1).cuda().contiguous(),
                           dev_i32(np.arange(B + 1) * n), zero, self.table)

    def query(self, rows):
        q = torch.zeros((rows, self.Hq, self.D), dtype=self.ctx.torch_dtype, device="cuda")
        q[:, :, 0] = 1.0
        return q

    def decode(self, bound=0):
        out = torch.full((self.B, self.Hq, self.D), float("nan"), dtype=self.ctx.torch_dtype, device="cuda")
        self.ctx.attn_decode(self.query(self.B), self.kc, self.vc, self.table, self.lens, out, bound or self.n)
        return out.double().cpu()

    def decode_by_slices(self):
        """With a bound of 1000 tokens, beyond what is decoded whole."""
        return self.decode(1000)

    def prefill(self):
        """The last position of every sequence (which sees all its keys), as decode returns it."""
        T = self.B * self.new
        out = torch.full((T, self.Hq, self.D), float("nan"), dtype=self.ctx.torch_dtype, device="cuda")
        self.ctx.attn_prefill(self.query(T), self.kc, self.vc, dev_i32(np.arange(self.B + 1) * self.new), self.before, self.table, out,
                              max_q_len=self.new)
        return out.double().cpu()[self.new - 1::self.new]

    def ways(self):
        """(name, result) of every kernel that serves this layout."""
        # (bf16, 128) prefill is another kernel, with another way of holding its weights
        names = ["decode", "decode_by_slices"] if (self.dtype, self.D) == ("bf16", 128) else ["decode", "prefill"]
        for plain in (0, 1):
            self.ctx.set_option(binding.OPT_FORCE_PLAIN, plain)
            for name in names:
                yield name + (", plain" if plain else ""), getattr(self, name)()
        self.ctx.close()


def _both_prefills(**kw):
    """One sequence (its keys shared out among the wavefronts), and ninety short chunks (their rows are)."""
    return [Scored(**kw), Scored(**kw, B=90, before=len(kw["log2_w"]) - 3)]


@pytest.mark.parametrize("dtype,D,Hkv", LAYOUTS, ids=IDS)
def test_large_values_do_not_overflow_the_sums(dtype, D, Hkv):
    """Values of 2^120 under 64 weights of 1 and 256 of 2^-7.5: sums of 2^126.03, if the weights are taken relative to the row's
    maximum.  The larger scores are keys 128..191, neither a wavefront's first nor its last block, and within what the
    exponent offset may lag behind the maximum."""
    log2_w = np.r_[np.zeros(128), np.full(64, 7.5), np.zeros(128)]
    values = np.full((320, D), 2.0 ** 120)
    for s in _both_prefills(dtype=dtype, D=D, Hkv=Hkv, log2_w=log2_w, values=values):
        for name, got in s.ways():
            say(f"{dtype}, head size {D}, {s.B} sequences, {name}: {got.min():.4g} .. {got.max():.4g}")
            # the mean of equal values: fp32 sums of 320 terms are within 320 2^-24, rounding to bf16 is 2^-9
            assert ((got / 2.0 ** 120 - 1).abs() <= (2.0 ** -8 if dtype == "bf16" else 320 * 2.0 ** -24)).all(), name


@pytest.mark.parametrize("dtype,D,Hkv", LAYOUTS[:2], ids=IDS[:2])
def test_weights_below_the_normal_numbers_count(dtype, D, Hkv):
    """One key of weight 1 and value 0, nineteen of weight 2^-128 and value 2^125: 19 / 8, not 0."""
    log2_w = np.r_[0.0, np.full(19, -128.0)]
    values = np.r_[np.zeros((1, D)), np.full((19, D), 2.0 ** 125)]
    for s in _both_prefills(dtype=dtype, D=D, Hkv=Hkv, log2_w=log2_w, values=values):
        for name, got in s.ways():
            say(f"{dtype}, head size {D}, {s.B} sequences, {name}: {got.min():.6g} .. {got.max():.6g} (19/8 = 2.375)")
            assert ((got - 2.375).abs() <= 1e-5).all(), name    # (exact in bf16; powers of two and small sums in fp32)


@pytest.mark.parametrize("dtype,D,Hkv", LAYOUTS[:2], ids=IDS[:2])
def test_weights_have_the_bits_of_fp32(dtype, D, Hkv):
    """Values that cancel to 2^-16 of their size: what is left tells weights of 24 bits from weights of 16.  (A weight of 24 bits:
    products exact to 2^-24 of terms of size 4 at most, exponents good to 2^-23: together 0.1 of what is left, by the 2-norm;
    weights of 16 bits measured 0.47.)"""
    rng = np.random.default_rng(1)
    bf = lambda x: torch.as_tensor(x).to(torch.bfloat16).double().numpy()
    n = 48
    a = rng.integers(-32, 1, size=n)
    a[-3:] = (-9, -20, -13)
    w = 2.0 ** (a / 8)
    values = bf(rng.standard_normal((n, D)))
    values[n - 2:] = 0
    for j in (n - 2, n - 1):       # each takes away what the sum over the keys before it comes to, as far as bf16 can
        values[j] = bf(-(w[:j, None] * values[:j]).sum(0) / w[j])
    want = torch.as_tensor((w[:, None] * values).sum(0) / w.sum())
    for s in _both_prefills(dtype=dtype, D=D, Hkv=Hkv, log2_w=a / 8, values=values):
        for name, got in s.ways():
            err = float(((got - want).norm(dim=-1) / want.norm()).max())
            say(f"{dtype}, head size {D}, {s.B} sequences, {name}: off by {err:.3f} of what the sums leave")
            assert err <= 0.2, name


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("bf16", 64)], ids=["f32-d64", "bf16-d64"])
def test_slices_whose_scores_are_all_minus_infinity(dtype, D):
    """Decode in slices of 64 tokens whose first 64 (a whole round of the merge) or 65 hold nothing but scores of minus
    infinity: they weigh nothing, and the result is that of the keys behind them."""
    for dead in (64, 65):
        n = dead * 64 + 70
        log2_w = np.r_[np.full(dead * 64, -np.inf), np.zeros(70)]
        values = np.r_[np.ones((dead * 64, D)), np.full((70, D), 3.0)]
        s = Scored(dtype, D, 2, log2_w, values)
        s.ctx.set_option(binding.OPT_DECODE_SPLIT_TOKENS, 64)
        got = s.decode()
        say(f"{dtype}, head size {D}, {dead} slices of minus infinity of {(n + 63) // 64}: {got.min():.6g} .. {got.max():.6g}")
        assert ((got - 3.0).abs() <= 1e-5).all()
        s.ctx.close()
