"""Decode of (bf16, head size 128) batches of short contexts (decode_short_kernel): on the host, that each case below gets the
wavefronts it is listed for; on the GPU, against the fp64 CPU oracle in a cache whose unwritten slots are not numbers, with lengths at
the edges of blocks and of the wavefronts' rounds, sequences that are empty, query and new rows that are slices of wider ones, called twice and with the
append fused in: the same bits, and the cache bit for bit the oracle's."""
import os
import subprocess

import numpy as np
import pytest

from paper_2504_18154_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _ragged(B, most, seed=81):
    n = wl.rng_for(seed).integers(1, most + 1, size=B)
    n[0] = most
    return n.tolist()


# name, heads, lengths, wavefronts per (sequence, K/V head) (0: another kernel has the batch), the caller's bound where it is not the longest
CASES = [("one-block", (40, 8), [1, 15, 16, 2], 1), ("two-blocks", (8, 1), [17, 31, 32, 1, 16], 1), ("one-many", (52, 52), _ragged(40, 32), 1),
         ("two", (5, 1), [33, 48, 64, 65, 96, 1, 80, 95], 2), ("two-many", (40, 8), _ragged(130, 384), 2), ("two-G16", (16, 1), _ragged(600, 200), 2),
         ("four", (64, 8), [384, 97, 383, 1, 17, 130], 4), ("four-one-sequence", (3, 3), [512], 4), ("four-most", (40, 8), _ragged(36, 640), 4),
         ("four-many", (32, 8), _ragged(90, 1152), 4), ("four-very-many", (8, 8), _ragged(200, 1024), 4),
         # more workgroups than CUs, handed out by length: groups of 33 and 32 sequences, more ids than a register holds, and with more than 4096
         # (sequence, K/V head)s, whose blocks are written past the caches
         ("four-two-groups", (16, 4), _ragged(65, 400), 4), ("four-windows", (8, 8), [60, 4300, 4096, 4097, 2049] + _ragged(96, 60), 4, 1600),
         ("one-stream", (8, 8), _ragged(520, 128), 1), ("two-stream", (16, 8), [17, 530, 600] + _ragged(517, 40), 2),
         ("two-stream-most", (8, 8), _ragged(510, 30) + [33, 825, 832], 2),
         ("slices", (40, 8), [513], 0), ("persistent", (52, 52), [1300] * 128, 0),
         # one long context among short ones: its walk would be the launch (us in balanced slices or by the persistent kernel / whole: 15.3 / 21.3,
         # 15.5 / 19.9, 10.7 / 13.2, 60.7 / 69.2)
         ("ragged-64x8", (64, 8), [1703] + [497] * 16, 0), ("ragged-32x8", (32, 8), [1562] + [550] * 17, 0), ("ragged-52x52", (52, 52), [823, 102, 102], 0),
         ("ragged-40x8", (40, 8), [3668] + [980] * 64, 0)]


def _bound(case):
    return case[4] if len(case) > 4 else max(case[2])


def test_each_case_gets_the_wavefronts_it_is_listed_for(tmp_path):
    calls = ", ".join(f"decode_short({len(c[2])}, {c[1][1]}, {_bound(c)}, 256)" for c in CASES)
    src, exe = tmp_path / "waves.cpp", tmp_path / "waves"
    src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "decode_slices.h"\nint main() { for (int w : {%s}) std::printf("%%d ", w); }'
                   % calls.replace("decode_short", "eco::decode_short"))
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2504_18154_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split() == [str(c[3]) for c in CASES]


@pytest.mark.gpu
@pytest.mark.parametrize("case", [c for c in CASES if c[3]], ids=lambda c: c[0])
def test_against_the_oracle(case):
    import torch

    from paper_2504_18154_amd import binding
    from tests.parity_util import Layer, compare, compare_lse, dev_i32, say
    name, heads, lens = case[:3]
    bound = _bound(case)
    Hq, Hkv = heads
    model = wl.ModelShape("short", Hq, Hkv, 128, 1, "bf16")
    lens = np.asarray(lens, dtype=np.int32)
    say(f"decode, {name}, heads {heads}, {len(lens)} sequences up to {lens.max()} tokens")
    pb = wl.prefill_batch(model, lens, 55)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v = (wl.randn((pb.T, Hkv, 128), "bf16", s) for s in (1, 2))
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, Hq, 128), "bf16", 3)
    ref, ref_lse = layer.decode_oracle(q, pb.block_table, lens)
    out, lse = layer.decode_gpu(q, pb.block_table, lens, bound)
    compare("decode", out, ref, "bf16")
    compare_lse("decode", lse, ref_lse, "bf16")
    last = torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)
    wide = torch.full((pb.B, Hq + 2 * Hkv, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide[:, :Hq], wide[:, Hq:Hq + Hkv], wide[:, Hq + Hkv:] = q.cuda(), k[last].cuda(), v[last].cuda()
    for kn, vn, qs in ((k[last].cuda(), v[last].cuda(), q.cuda()), (wide[:, Hq:Hq + Hkv], wide[:, Hq + Hkv:], wide[:, :Hq])):
        fused, fused_lse = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
        layer.wipe_newest(pb.block_table, lens)
        layer.ctx.attn_decode_append(qs, kn, vn, layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), fused, bound, fused_lse)
        torch.cuda.synchronize()
        assert torch.equal(fused, out) and torch.equal(fused_lse, lse), "the fused append changes the result"
        layer.assert_cache_bit_exact()
    no = torch.full_like(out, float("nan"))
    assert binding.attn_decode_noalloc(layer.ctx.layout, q.cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), no, bound) == binding.OK
    torch.cuda.synchronize()
    assert torch.equal(no, out), "the call without a context differs"
    # empty sequences have no output and cost their neighbours nothing
    some = lens.copy()
    some[1::2] = 0
    holes = torch.full_like(out, 7.0)
    layer.ctx.attn_decode(q.cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(some), holes, bound)
    torch.cuda.synchronize()
    assert torch.equal(holes[::2], out[::2]) and (holes[1::2] == 7.0).all()
    layer.close()


@pytest.mark.gpu
@pytest.mark.parametrize("L", [30, 90, 200], ids=["one", "two", "four"])
def test_infinite_values_reach_only_their_own_elements(L):
    """Infinite V elements, one of them in the token that the fused append brings: infinite there, and what it was elsewhere (the remainder
    of a weight may be zero, and must not make them NaN)."""
    import torch

    from tests.parity_util import Layer, dev_i32
    model = wl.ModelShape("short", 40, 8, 128, 1, "bf16")
    lens = np.asarray([L, 7], dtype=np.int32)
    pb = wl.prefill_batch(model, lens, 57)
    layer = Layer(model, pb.num_blocks, pb.B, pb.block_table.shape[1])
    k, v = (wl.randn((pb.T, 8, 128), "bf16", s) for s in (1, 2))
    k = k * 3  # (weights of a few keys are close to one, of others to zero)
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    q = wl.randn((pb.B, 40, 128), "bf16", 3)
    out, _ = layer.decode_gpu(q, pb.block_table, lens)
    v[2, :, 5] = float("inf")
    v[L - 1, :, 100] = float("inf")
    layer.append(k, v, pb.cu_q, pb.ctx_before, pb.block_table)
    last = torch.as_tensor(pb.cu_q[1:] - 1, dtype=torch.long)
    got = torch.full_like(out, float("nan"))
    layer.wipe_newest(pb.block_table, lens)
    layer.ctx.attn_decode_append(q.cuda(), k[last].cuda(), v[last].cuda(), layer.kc, layer.vc, dev_i32(pb.block_table), dev_i32(lens), got, int(lens.max()))
    torch.cuda.synchronize()
    layer.assert_cache_bit_exact()
    assert torch.isinf(got[0, :, [5, 100]]).all() and torch.isfinite(got[1]).all()
    others = [d for d in range(128) if d not in (5, 100)]
    assert (got[0][:, others].float() - out[0][:, others].float()).abs().max() <= 2.0 ** -8 * 4  # (a bf16 spacing of values up to 4)
    layer.close()
