"""M in FP32 with a cell a thread: at most 64 vector registers in every shape.
Up to there two workgroups of 1024 threads (eight wavefronts a SIMD) share a
compute unit; with two registers more one does, and a call at L = 62 or 64 took
a tenth longer.  Read from the compiler's own figures."""
import os
import re
import subprocess

import pytest

from paper_2508_16298_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_two_wide_workgroups_fit(tmp_path):
    r = subprocess.run([build.HIPCC, *build.CFLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(build.CSRC, "lattice.hip"), "-o", str(tmp_path / "lattice.o")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    # _ZN2qh9k_apply_MIfLi1E...: R = float, MC = 1
    regs = {b.split()[0]: (int(re.search(r" VGPRs: (\d+)", b)[1]), int(re.search(r"ScratchSize[^:]*: (\d+)", b)[1]))
            for b in r.stderr.split("Function Name: ")[1:] if b.startswith("_ZN2qh9k_apply_MIfLi1E")}
    assert len(regs) == 6
    assert all(v <= 64 and s == 0 for v, s in regs.values()), regs
