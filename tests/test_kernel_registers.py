"""What the compiler reports of the small-batch decode kernels, of the one for whole contexts and of the prefill kernel for short
contexts: none of their instances goes through scratch memory (fp32 heads of 256 elements fill the registers; spilled, a call of 50
tokens took 12.2 us instead of 10.6; the other two are within a few registers of what their wavefronts per SIMD leave them)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_18154_amd import build


def _scratch_and_spills(tmp_path, source):
    """{kernel: [scratch bytes per lane, registers spilled]} of a source."""
    hipcc = build._hipcc()
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    cmd = [hipcc, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-I", build.INCLUDE, "-c",
           os.path.join(build.CSRC, source), "-o", str(tmp_path / "any.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    of = {}
    for line in r.stderr.splitlines():
        if m := re.search(r"Function Name: (\S+)", line):
            name = m.group(1)
        elif m := re.search(r"(ScratchSize \[bytes/lane\]|VGPRs Spill): (\d+)", line):
            of.setdefault(name, []).append(int(m.group(2)))
    return of


def _assert_none(of, kernel, least):
    found = {n: v for n, v in of.items() if kernel in n}
    assert len(found) >= least and all(len(v) == 2 for v in found.values()), found
    assert all(v == [0, 0] for v in found.values()), {n: v for n, v in found.items() if v != [0, 0]}


def test_decode_kernels_do_not_spill(tmp_path):
    of = _scratch_and_spills(tmp_path, "attn_any_mfma.hip")
    _assert_none(of, "decode_any_kernel", 12)
    _assert_none(of, "decode_short_kernel", 6)


def test_prefill_kernel_for_short_contexts_does_not_spill(tmp_path):
    _assert_none(_scratch_and_spills(tmp_path, "attn_prefill_short.hip"), "prefill_short_kernel", 3)
