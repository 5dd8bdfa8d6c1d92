"""pme_forward_noalloc near its scratch limit on pencil meshes: calls whose workspace fits
with less than a KiB to spare work, and equal a plan's forward; calls a little past the limit
are refused before anything runs."""
import ctypes

import numpy as np
import pytest
import torch

import synth
from test_zz_no_alloc import _desc, _noalloc, _plan_forward

pytestmark = pytest.mark.gpu


def _frame(mesh, n):
    rng = np.random.default_rng(sum(mesh) + n)
    box = np.diag([0.9 * m for m in mesh])
    return synth.Frame(pos=rng.uniform(0, 1, (n, 3)) @ box, q=rng.normal(0, 1, n),
                       mu=rng.normal(0, 0.1, (n, 3)), box=box)


@pytest.mark.parametrize("mesh,p,n", [((30, 108, 1024), 6, 5000), ((60, 128, 450), 4, 50000)])
def test_accepted(mesh, p, n):
    print(f"case: {mesh} p={p} n={n}", flush=True)
    f = _frame(mesh, n)
    got, ref = _noalloc(f, mesh, p, 0.4), _plan_forward(f, mesh, p, 0.4)
    for k in ref:
        assert torch.equal(got[k], ref[k]), k


@pytest.mark.parametrize("mesh,p,n", [((36, 600, 128), 5, 1000), ((12, 800, 384), 4, 1),
                                      ((5, 720, 750), 6, 100000)])
def test_refused(mesh, p, n):
    from paper_2606_01598_amd import _lib
    x = torch.zeros(3 * n, device="cuda")
    e = torch.zeros(9, dtype=torch.float64, device="cuda")
    d = _desc(mesh, p, 0.4)
    rc = _lib.load().pme_forward_noalloc(ctypes.byref(d), torch.cuda.current_stream().cuda_stream, n,
                                         x.data_ptr(), None, None, e.data_ptr(), e.data_ptr(), None,
                                         None, None)
    assert rc == _lib.PME_ESCRATCH
