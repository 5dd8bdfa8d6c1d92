"""Positions that are not finite reach the outputs of the pair and feature kernels: every
atom in the cells around the one they are sorted into gets NaN (a feature in the channels of
the atom's species alone).  The cells have at most three along an axis, so that every other
atom is a candidate."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev, f32

pytestmark = pytest.mark.gpu
N, SIDE, BAD = 70, 16.0, 9


def _case(value):
    rng = np.random.default_rng(2)
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=dev())   # noqa: E731
    pos = rng.uniform(0.0, SIDE, (N, 3))
    pos[BAD, 1] = value
    q = np.where(np.arange(N) % 2, 1.0, -1.0)
    return t(pos), t(q), t(rng.normal(0, 0.3, (N, 3))), t(rng.uniform(0.2, 3.0, N)), t, rng


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_pair_kernels(value):
    from paper_2606_01598_amd.pme import Plan
    from paper_2606_01598_amd.pol import PolPlan
    pos, q, mu, pol, t, rng = _case(value)
    plan = PolPlan(np.eye(3) * SIDE, 0.35, 7.0, max_atoms=N)
    out = plan.real(pos, q, mu, pol, dE_dq=True)
    out["mixed"] = plan.mixed(pos, q, mu, pol, t(rng.normal(0, 1, (N, 3))))
    for k, x in out.items():
        assert bool(torch.isnan(x).all()), k
    box = torch.tensor(np.eye(3) * SIDE, device=dev())
    pme = Plan((18, 18, 18), 6, 0.35, max_atoms=N)
    model = plan.model(pme, pos, q, mu, pol, box)
    for k, x in model.items():
        assert bool(torch.isnan(x).all()), k


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_feature_kernels(value):
    from paper_2606_01598_amd.dip import DipPlan
    pos, q, _, _, t, rng = _case(value)
    plan = DipPlan(np.eye(3) * SIDE, N, cutoff=5.0)
    feat, vec = plan.features(pos, q)
    fd, vd = plan.features_jvp(pos, q, vec, t(rng.normal(0, 1, (N, 3))))
    theta = t(f32(synth.mlp_init(5, last_scale=1.0)))
    g = plan.position_vjp(theta, pos, q, feat, vec, t(rng.normal(0, 1, (N, 3))))
    assert bool(torch.isnan(g).all())
    rest = torch.arange(N, device=dev()) != BAD
    own = 0 if float(q[BAD]) > 0 else 1         # channels 8 own .. 8 own + 7 of each kind
    for k, x in (("feat", feat[:, :16]), ("squares", feat[:, 16:32]), ("vec", vec),
                 ("feat_dot", fd[:, :16]), ("squares_dot", fd[:, 16:32]), ("vec_dot", vd)):
        assert bool(torch.isnan(x[BAD]).all()), k
        assert bool(torch.isnan(x[rest][:, 8 * own:8 * own + 8]).all()), k
        assert bool(torch.isfinite(x[rest][:, 8 - 8 * own:16 - 8 * own]).all()), k
    assert bool(torch.isfinite(feat[:, 32:]).all()) and bool((fd[:, 32:] == 0).all())


@pytest.mark.parametrize("where", ["pos", "q", "mu"])
def test_solve_reports_residuals_that_are_not_finite(where):
    from paper_2606_01598_amd import _lib
    from paper_2606_01598_amd.pme import Plan
    from paper_2606_01598_amd.pol import PolPlan
    pos, q, mu, pol, _, _ = _case(float("nan") if where == "pos" else 3.0)
    if where == "q":
        q[BAD] = float("nan")
    if where == "mu":
        mu[BAD, 0] = float("nan")
    box = torch.tensor(np.eye(3) * SIDE, device=dev())
    pme = Plan((18, 18, 18), 6, 0.35, max_atoms=N)
    plan = PolPlan(box, 0.35, 7.0, max_atoms=N, warm_start=where == "mu")
    with pytest.raises(_lib.PMEError) as err:
        plan.scf(pme, pos, q, pol, box, tol=1e-6, max_iter=20, mu=mu)
    assert err.value.code == _lib.PME_ENONFINITE
