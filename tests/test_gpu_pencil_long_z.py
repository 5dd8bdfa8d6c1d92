"""The z passes of the pencil layout on long axes, where fewer pairs of rows than eight go
in a workgroup: lengths in more than two stages that take two to seven, odd row counts among
them.  Compared as in test_gpu_pencil."""
import pytest

from test_gpu_pencil import test_potential_matches_fft as potential_matches_fft

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh", [(5, 45, 625), (6, 20, 1024), (4, 54, 405), (5, 27, 972), (2, 40, 540)],
                         ids=lambda m: "x".join(map(str, m)))
def test_potential(mesh):
    potential_matches_fft(mesh)
