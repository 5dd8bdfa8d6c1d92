"""Host check of the two-stage line transforms of the pencil passes (csrc/fft_radix.h):
the wide register DFTs and every length up to 400 that splits into two of them, in both
orders of the radices, against a direct double-precision DFT."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("twostage") / "check")
    subprocess.run([HIPCC, "--offload-host-only", "-x", "hip", "-std=c++17", "-O2",
                    os.path.join(HERE, "fft_two_stage_check.hip"), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return [line.split() for line in out.splitlines()]


def test_wide_dfts_match_direct(report):
    rows = [r for r in report if r[0] == "dft"]
    assert {int(r[1]) for r in rows} == {2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20}
    for r in rows:
        assert float(r[3]) < 2e-6, r


def test_two_stage_lines_match_direct(report):
    rows = [r for r in report if r[0] == "two"]
    by_n = {int(r[1]): (int(r[2]), int(r[3])) for r in rows}
    assert by_n[320] == (20, 16) and by_n[160] == (16, 10) and by_n[4] == (2, 2)
    assert not {2, 3, 5, 125, 250, 243} & set(by_n)
    for r in rows:
        assert int(r[2]) * int(r[3]) == int(r[1]) and float(r[5]) < 1e-5, r
