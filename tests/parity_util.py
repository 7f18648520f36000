"""Shared plumbing of the GPU parity tests: run one layer's cache through both the HIP
library (via the C ABI binding) and the CPU oracle on the same seeded inputs."""
from __future__ import annotations

import sys

import numpy as np
import torch

from oracle import oracle as orc
from paper_2504_18154_amd import workloads as wl

# Tolerances (outputs, GPU vs fp64 oracle).  bf16 inputs, fp32 accumulation: the stated
# bar.  fp32: derived from fp32 accumulation over a few hundred keys plus exp2 error,
# with two orders of magnitude of headroom.
TOL = {"bf16": (1e-2, 1e-3), "f32": (1e-4, 1e-5)}
# log-sum-exp (natural log): 1e-3 where the row sum is taken in fp32 (decode, the plain
# kernels).  The matrix-core prefill kernel sums the bf16-rounded weights (the same values
# the second product consumes, so numerator and denominator of the output agree).  A bf16
# number has 8 significant bits: rounding to nearest moves a weight by at most half a
# spacing, which relative to a value just above a power of two is 2^-8 = 3.9e-3.  With a
# flat softmax the roundings of hundreds of weights average out (errors of 1e-4 in the
# tests); with near one-hot weights the row sum is one weight and carries its full rounding
# error, so 2^-8 is the bound on the relative error of the sum and hence on the error of its
# log: 4e-3 there (`bf16_row_sum=True`) and nowhere else.
LSE_TOL = {"bf16": 1e-3, "f32": 1e-4}
LSE_TOL_BF16_ROW_SUM = 4e-3
# Full-size workloads: at most this share of the output elements may miss the stated 1e-2
# and rely on the bound for coarse bf16 outputs (see compare).
MAX_RELAXED_SHARE = 1e-4


def say(msg: str):
    print(msg, flush=True)
    sys.stdout.flush()


def dev_i32(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.int32), device="cuda")


class Layer:
    """One layer's paged cache held twice: by the HIP library (device) and by the oracle (host)."""

    def __init__(self, model: wl.ModelShape, num_blocks: int, max_batch: int, max_blocks_per_seq: int,
                 oracle_cache: bool = True):
        from paper_2504_18154_amd import binding
        self.model = model
        self.ctx = binding.Context(model.Hq, model.Hkv, model.D, num_blocks, model.dtype, max_batch,
                                   max_blocks_per_seq)
        self.kc, self.vc = self.ctx.new_cache()
        dt = orc.BF16 if model.dtype == "bf16" else orc.F32
        self.shape = orc.Shape(model.Hq, model.Hkv, model.D, model.bs, num_blocks, dt)
        if oracle_cache:
            self.okc, self.ovc = orc.new_cache(self.shape)

    def append(self, k_new: torch.Tensor, v_new: torch.Tensor, cu_q, ctx_before, table, max_new_len=None):
        """k_new/v_new: tensors on any device; the same bits go to both sides."""
        kd, vd = k_new.cuda(), v_new.cuda()
        self.ctx.kv_append(self.kc, self.vc, kd, vd, dev_i32(cu_q), dev_i32(ctx_before), dev_i32(table),
                           max_new_len=max_new_len)
        orc.kv_append(self.shape, self.okc, self.ovc, wl.to_bits(k_new), wl.to_bits(v_new), cu_q, ctx_before, table)

    def wipe_newest(self, table, ctx_len):
        """Overwrites the last token of every sequence with NaN rows in the device's cache (and not in the oracle's): what a
        fused append has to bring back."""
        n = len(ctx_len)
        wipe = torch.full((n, self.model.Hkv, self.model.D), float("nan"), dtype=self.kc.dtype, device="cuda")
        self.ctx.kv_append(self.kc, self.vc, wipe, wipe, dev_i32(np.arange(n + 1)), dev_i32(np.asarray(ctx_len) - 1), dev_i32(table),
                           max_new_len=1)

    def assert_cache_bit_exact(self):
        torch.cuda.synchronize()
        gk = wl.to_bits(self.ctx.k_logical(self.kc))
        gv = wl.to_bits(self.ctx.v_logical(self.vc))
        if self.model.dtype == "f32":
            assert np.array_equal(gk.view(np.uint32), self.okc.view(np.uint32)), "K pool differs from the oracle's"
            assert np.array_equal(gv.view(np.uint32), self.ovc.view(np.uint32)), "V pool differs from the oracle's"
        else:
            assert np.array_equal(gk, self.okc), "K pool differs from the oracle's"
            assert np.array_equal(gv, self.ovc), "V pool differs from the oracle's"

    def prefill_gpu(self, q: torch.Tensor, cu_q, ctx_before, table, max_q_len=None):
        qd = q.cuda()
        out = torch.full_like(qd, float("nan"))
        lse = torch.full(qd.shape[:2], float("nan"), dtype=torch.float32, device="cuda")
        if max_q_len is None:
            max_q_len = int(np.max(np.diff(cu_q))) if len(cu_q) > 1 else 0
        self.ctx.attn_prefill(qd, self.kc, self.vc, dev_i32(cu_q), dev_i32(ctx_before), dev_i32(table), out, lse,
                              max_q_len=max_q_len)
        torch.cuda.synchronize()
        return out, lse

    def decode_gpu(self, q: torch.Tensor, table, ctx_len, max_ctx_len=None):
        qd = q.cuda()
        out = torch.full_like(qd, float("nan"))
        lse = torch.full(qd.shape[:2], float("nan"), dtype=torch.float32, device="cuda")
        if max_ctx_len is None:
            max_ctx_len = int(np.max(ctx_len))
        self.ctx.attn_decode(qd, self.kc, self.vc, dev_i32(table), dev_i32(ctx_len), out, max_ctx_len, lse)
        torch.cuda.synchronize()
        return out, lse

    def prefill_oracle(self, q, cu_q, ctx_before, table):
        return orc.attn_prefill(self.shape, wl.to_bits(q), self.okc, self.ovc, cu_q, ctx_before, table)

    def decode_oracle(self, q, table, ctx_len):
        return orc.attn_decode(self.shape, wl.to_bits(q), self.okc, self.ovc, table, ctx_len)

    def close(self):
        self.ctx.close()


def bf16_ulp(x: np.ndarray) -> np.ndarray:
    """Spacing of bf16 numbers (8 significant bits) at |x|."""
    ax = np.maximum(np.abs(x), 2.0 ** -126)
    return 2.0 ** (np.floor(np.log2(ax)) - 7)


def compare(name, got: torch.Tensor, ref: np.ndarray, dtype: str, rows=None, max_relaxed_share=None):
    """max-abs and mean-abs error of GPU output vs the fp64 oracle.

    bf16 outputs: the stated bounds are 1e-2 max-abs and 1e-3 mean-abs.  A bf16 number
    with |o| >= 2 has spacing >= 2^-6 > 1e-2, so rounding the exact result to the output type
    alone can miss it by half a spacing (0.0078 for |o| < 4, 0.0156 for |o| < 8), and the
    bf16 rounding of the weights before the second product adds up to 2^-9 |o|.  Elements
    with |o| >= 2 (short contexts, where the output is close to a single large V entry) are
    therefore held to max(1e-2, half a spacing + 2^-9 |o|); everything else to 1e-2.  The
    number of elements that actually miss 1e-2 is printed and, with `max_relaxed_share`
    (the full-size workloads), bounded as a share of all elements."""
    if rows is not None:   # select on the device first: full outputs can be gigabytes
        got = got[torch.as_tensor(np.asarray(rows), dtype=torch.long, device=got.device)]
    g = got.detach().double().cpu().numpy()
    assert g.shape == ref.shape, (g.shape, ref.shape)
    assert np.all(np.isfinite(g)), f"{name}: non-finite values in the GPU output"
    err = np.abs(g - ref)
    mx, mean = float(err.max()) if err.size else 0.0, float(err.mean()) if err.size else 0.0
    tmax, tmean = TOL[dtype]
    bound = np.full(ref.shape, tmax)
    coarse = relaxed = 0
    if dtype == "bf16":
        big = np.abs(ref) >= 2.0
        bound = np.where(big, np.maximum(tmax, 0.5 * bf16_ulp(ref) + 2.0 ** -9 * np.abs(ref)), tmax)
        coarse = int(big.sum())
        relaxed = int((err > tmax).sum())
    worst = float((err / bound).max()) if err.size else 0.0
    say(f"  {name}: max-abs {mx:.3e} (<= {tmax:g}; {coarse} of {ref.size} elements have |o| >= 2, {relaxed} miss "
        f"{tmax:g} and are held to half a bf16 spacing + 2^-9 |o|; worst err/bound {worst:.2f})  "
        f"mean-abs {mean:.3e} (<= {tmean:g})")
    assert np.all(err <= bound) and mean <= tmean, f"{name}: max-abs {mx:.3e}, mean-abs {mean:.3e}, worst {worst:.2f}"
    if max_relaxed_share is not None:
        assert relaxed <= max_relaxed_share * ref.size, \
            f"{name}: {relaxed} of {ref.size} elements miss {tmax:g} (more than a share of {max_relaxed_share:g})"
    return mx, mean


def compare_lse(name, got: torch.Tensor, ref: np.ndarray, dtype: str, rows=None, bf16_row_sum=False):
    """`bf16_row_sum`: the result comes from the matrix-core prefill kernel (see LSE_TOL)."""
    if rows is not None:
        got = got[torch.as_tensor(np.asarray(rows), dtype=torch.long, device=got.device)]
    g = got.detach().double().cpu().numpy()
    tol = LSE_TOL_BF16_ROW_SUM if bf16_row_sum and dtype == "bf16" else LSE_TOL[dtype]
    err = float(np.abs(g - ref).max()) if ref.size else 0.0
    say(f"  {name}: lse max-abs {err:.3e} (<= {tol:g})")
    assert err <= tol, f"{name}: lse error {err:.3e}"
