"""Registers of the batched matrix-core operator (compiled here for gfx950, no
GPU): the waves per SIMD that its LDS allows, three up to N = 7 and two at
N = 8, and no vector register in scratch memory.  With the direction formed at
the gather N = 6 fell to two and N = 8 to one."""
import os
import re
import subprocess

import pytest

from paper_1403_0968_amd import build


def test_batched_operator_waves_per_simd(tmp_path):
    try:
        hipcc = build._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    src = os.path.join(build.CSRC, "ax_mfma.hip")
    r = subprocess.run([hipcc, *build.COMMON, "-x", "hip", "--cuda-device-only", "-c", src, "-o",
                        str(tmp_path / "x.o"), "-Rpass-analysis=kernel-resource-usage"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    use = {}
    for line in r.stderr.splitlines():
        m = re.search(r"remark: +([A-Za-z][^:]*): (\S+)", line)
        if m and m.group(1) == "Function Name":
            cur = use.setdefault(m.group(2), {})
        elif m:
            cur[m.group(1)] = m.group(2)
    got = {n: u for n, u in use.items() if "k_bax_mfma" in n}
    assert len(got) == 16  # orders 1 to 8, with and without the split of D
    for n, u in got.items():
        want = 2 if "k_bax_mfma9" in n else 3
        assert int(u["Occupancy [waves/SIMD]"]) >= want, (n, u)
        assert int(u["VGPRs Spill"]) == 0, (n, u)
