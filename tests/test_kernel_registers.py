"""What the compiler reports of the small-batch decode kernels: none of their instances goes through scratch memory (fp32 heads of
256 elements fill the registers; spilled, a call of 50 tokens took 12.2 us instead of 10.6)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_18154_amd import build


def test_decode_kernels_do_not_spill(tmp_path):
    hipcc = build._hipcc()
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    cmd = [hipcc, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-I", build.INCLUDE, "-c",
           os.path.join(build.CSRC, "attn_any_mfma.hip"), "-o", str(tmp_path / "any.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    of = {}
    for line in r.stderr.splitlines():
        if m := re.search(r"Function Name: (\S+)", line):
            name = m.group(1)
        elif m := re.search(r"(ScratchSize \[bytes/lane\]|VGPRs Spill): (\d+)", line):
            of.setdefault(name, []).append(int(m.group(2)))
    decode = {n: v for n, v in of.items() if "decode_any_kernel" in n}
    assert len(decode) >= 12 and all(len(v) == 2 for v in decode.values()), decode
    assert all(v == [0, 0] for v in decode.values()), {n: v for n, v in decode.items() if v != [0, 0]}
