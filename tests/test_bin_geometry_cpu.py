"""Host check of the bins and tiles of plans (csrc/geometry.h) over 5-smooth meshes, tile
targets, orders and spreads: the bounds that the gather (one thread a bin of its tile) and
the tile spread (bins it scans) count on, and bins that divide the tiles and the mesh."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def test_bins_keep_the_kernels_bounds(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "check")
    subprocess.run([HIPCC, "--offload-host-only", "-x", "hip", "-std=c++17", "-O2",
                    os.path.join(HERE, "bin_geometry_check.hip"), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    bad = [line for line in out if line.startswith("plan ")]
    assert not bad, (len(bad), bad[:8])
    counts = {k: int(v) for k, v in (line.split() for line in out)}
    assert counts["plans"] > 200000 and counts["planes"] > 50000
