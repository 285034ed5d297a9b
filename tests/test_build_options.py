"""The build's documented overrides compile (CPU: syntax and template instantiation only)."""
import os
import subprocess

import pytest


@pytest.mark.parametrize("flags", ["-DMFQ_BRICK_P4=4,1,2", "-DMFQ_BRICK_P1=8,4,2 -DMFQ_BRICK_P2=5,2,2 -DMFQ_BRICK_P8=1,1,2"])
def test_brick_shape_override_compiles(flags):
    from paper_1910_13247_amd import build
    src = os.path.join(build.CSRC, "kernels_cell.hip")
    r = subprocess.run([build.HIPCC, "-fsyntax-only", "-std=c++17", f"--offload-arch={build.ARCH}", "-I",
                        os.path.join(build.ROOT, "include"), "-x", "hip", *flags.split(), src], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
