"""The bins of the plane spreads (one cell wide in x) and the counted front end of the
gather where they can go wrong: an ionic crystal that fills every third x-plane, so that
bins pass their capacity and records overflow; a box whose atoms all lie in one tile of
the gather (many windows of its queue, and one window with a single atom more than the
queue holds); and a pair of atoms.  Against
the FP64 oracle, with the bounds of the other parity tests."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import (E_REL_TOL, RMS_REL_TOL, host, oracle_forward, oracle_hvp, rel, rms_rel,
                      to_dev)

pytestmark = pytest.mark.gpu


def _frame(kind, diag):
    rng = np.random.default_rng(sum(map(ord, kind)))
    diag = np.asarray(diag, dtype=float)
    if kind == "layered":
        g = np.stack(np.meshgrid(np.arange(0, diag[0], 3.0), np.arange(0, diag[1], 1.5),
                                 np.arange(0, diag[2], 1.5), indexing="ij"), -1).reshape(-1, 3)
        pos = g + rng.uniform(0.0, 0.2, g.shape)
    else:
        n = {"two": 2, "queue": 129, "tile": 700}[kind]
        pos = rng.uniform(0.5, 4.5, (n, 3))
    n = len(pos)
    q = rng.normal(0.0, 1.0, n)
    q -= q.mean()
    return synth.Frame(pos=pos, q=q, mu=rng.normal(0.0, 0.1, (n, 3)), box=np.diag(diag))


@pytest.mark.parametrize("kind,mesh,spread", [
    ("layered", (30, 32, 32), "fused"), ("layered", (24, 30, 45), "fused"),
    ("layered", (24, 128, 125), "band"), ("queue", (32, 32, 32), "fused"),
    ("tile", (32, 27, 25), "fused"), ("tile", (20, 135, 128), "band"),
    ("two", (16, 16, 16), "fused")])
def test_crowded_bins_and_tiles(kind, mesh, spread):
    from paper_2606_01598_amd.pme import Plan
    f = _frame(kind, mesh)
    print(f"case: {kind} n={f.n} mesh={mesh}", flush=True)
    alpha = 0.35
    plan = Plan(mesh, 6, alpha, max_atoms=f.n)
    assert plan.spread_kind == spread
    pos, q, mu, box = to_dev(f)
    v = synth.random_cotangents(f.n, 5, scale_r=0.1)
    ref = oracle_forward(f, mesh, 6, alpha, 1.0, with_q=True, with_mu=True)
    href = oracle_hvp(f, mesh, 6, alpha, v)
    vd = [torch.tensor(np.asarray(x), dtype=torch.float32, device=pos.device) for x in v]
    out = plan.forward(pos, q, mu, box)
    g = plan.backward(pos, q, mu, box, *vd)
    plan.status()
    assert rel(host(out["energy"]).sum(), ref.energy) <= E_REL_TOL
    for k in ("dE_dpos", "dE_dq", "dE_dmu"):
        assert rms_rel(host(out[k]), getattr(ref, k)) <= RMS_REL_TOL, k
    for k, want in zip(("g_pos", "g_q", "g_mu"), href):
        assert rms_rel(host(g[k]), want) <= RMS_REL_TOL, k


@pytest.mark.parametrize("p", [2, 3, 4, 5, 6, 7])
def test_gather_orders(p):
    """Both gathers and the step's for every number of lanes an atom has (with four and
    more its output vectors are stored by different lanes), some outputs left out."""
    from paper_2606_01598_amd.pme import Plan
    f = synth.molten_box(90, 40 + p, L=13.0)
    mesh, alpha = (16, 20, 18), 0.4
    v = synth.random_cotangents(f.n, p, scale_r=0.2, scale_mu=0.5)
    ref = oracle_forward(f, mesh, p, alpha, 1.0, with_q=True, with_mu=True)
    href = oracle_hvp(f, mesh, p, alpha, v)
    plan = Plan(mesh, p, alpha, max_atoms=f.n, concurrent=True)
    args = to_dev(f)
    vd = [torch.tensor(np.asarray(x), dtype=torch.float32, device=args[0].device) for x in v]
    want = {"dE_dpos": ref.dE_dpos, "dE_dq": ref.dE_dq, "dE_dmu": ref.dE_dmu,
            "g_pos": href[0], "g_q": href[1], "g_mu": href[2]}
    both = plan.step(*args, *vd)
    apart = {**plan.forward(*args), **plan.backward(*args, *vd)}
    less = plan.backward(*args, *vd, g_pos=False, g_q=False)
    plan.status()
    assert sorted(less) == ["g_mu"] and torch.equal(less["g_mu"], apart["g_mu"])
    for k, w in want.items():
        assert rms_rel(host(both[k]), w) <= RMS_REL_TOL, ("step", k)
        assert rms_rel(host(apart[k]), w) <= RMS_REL_TOL, k


@pytest.mark.parametrize("mesh,spread,opt", [((24, 20, 18), "fused", False), ((16, 30, 25), "fused", True),
                                             ((20, 128, 125), "band", False)])
def test_step_in_shared_launches_equals_two_streams(mesh, spread, opt):
    """pme_step puts both chains' passes into the same launches; with the launch timer
    armed for one of their kernels it runs them apart.  Every output is the same bit for
    bit, in either order on one plan and without some inputs."""
    from paper_2606_01598_amd.pme import Plan
    f = synth.molten_box(150, 11, L=15.0)
    plan = Plan(mesh, 6, 0.4, max_atoms=f.n, concurrent=True, optimal_influence=opt)
    assert plan.spread_kind == spread
    pos, q, mu, box = to_dev(f)
    v = [torch.tensor(x, dtype=torch.float32, device=pos.device)
         for x in synth.random_cotangents(f.n, 9, scale_r=0.1)]
    for args in ((pos, q, mu, box, *v), (pos, q, None, box, v[0], None, None),
                 (pos, None, mu, box, None, None, v[2])):
        runs = []
        for kind in (None, "spread", "fft_x", None, "gather_hvp"):
            plan.timer(kind)
            runs.append({k: x.clone() for k, x in plan.step(*args).items()})
        plan.timer(None)
        plan.status()
        for r in runs[1:]:
            assert all(torch.equal(r[k], runs[0][k]) for k in runs[0])
