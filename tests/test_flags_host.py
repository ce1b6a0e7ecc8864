"""The order flags of the first pass (lopc_tile.h, the same source the kernels
use) compiled for the host: no flag names a neighbour outside the grid, also for
infinities and products past the bin range at every face of the grid."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_no_flag_leaves_the_grid(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "host_flags")
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1",
                    "-std=c++17", "-ffp-contract=off", "-fno-fast-math", "-o", exe,
                    os.path.join(HERE, "host_flags.cpp")], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
