"""The hand-over between the workgroups of a whole step is written for gfx950: the
step kernels refuse to compile for another target rather than race on it."""
import os
import subprocess

import pytest

from paper_2508_18205_amd import build as B


@pytest.mark.parametrize("arch,good", [("gfx950", True), ("gfx942", False), ("gfx1200", False)])
def test_step_kernels_compile_for_gfx950_only(arch, good):
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    r = subprocess.run([hipcc, "-std=c++17", f"--offload-arch={arch}", "--cuda-device-only", "-E", "-I",
                        os.path.join(B.ROOT, "include"), os.path.join(B.CSRC, "step.hip"), "-o", os.devnull],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == good, r.stderr
    assert good or "gfx950 only" in r.stderr
