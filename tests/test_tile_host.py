"""The geometry of the repair's tiles (lopc_tile.h, the same source the kernels
use) compiled for the host: faces, blind cells and face steps of every tile
shape against the stencil itself."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_faces_cover_the_halo_of_every_tile_shape(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "host_tile")
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1",
                    "-std=c++17", "-o", exe, os.path.join(HERE, "host_tile.cpp")],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert r.stdout.count(" 0 mistakes") == 5
