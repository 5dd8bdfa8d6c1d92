"""pol_model and pol_model_hvp with outputs in the place of their inputs give what separate
buffers give.

Tolerance: the order of an atom's pairs differs from call to call (cells are filled by
atomics), which moves a sum of some 70 terms by a few 2^-24 of the largest: 1e-5 of the RMS.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, rms_rel

pytestmark = pytest.mark.gpu
N, SIDE = 300, 22.0
TOL = 1e-5


def _setup():
    from paper_2606_01598_amd.pme import Plan
    from paper_2606_01598_amd.pol import PolPlan
    rng = np.random.default_rng(6)
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=dev())   # noqa: E731
    x = {"pos": t(rng.uniform(0, SIDE, (N, 3))), "q": t(rng.normal(0, 1, N)),
         "mu": t(rng.normal(0, 0.3, (N, 3))), "pol": t(rng.uniform(0.2, 3.0, N)),
         "v_pos": t(rng.normal(0, 1, (N, 3))), "v_q": t(rng.normal(0, 1, N)),
         "v_mu": t(rng.normal(0, 1, (N, 3)))}
    box = torch.tensor(np.eye(3) * SIDE, device=dev())
    plan = PolPlan(box, 0.35, 8.0, max_atoms=N + 5)
    return plan, Plan((24,) * 3, 6, 0.35, max_atoms=N + 5), box, x


@pytest.mark.parametrize("g_q,g_mu", [("v_q", "v_mu"), ("q", "mu"), (None, "v_pos"), (None, "pos"),
                                      ("pol", None), ("shifted", None)])
def test_hvp(g_q, g_mu):
    plan, pme, box, x = _setup()
    call = lambda y, **kw: plan.model_hvp(pme, y["pos"], y["q"], y["mu"], y["pol"], box, y["v_pos"],   # noqa: E731
                                          y["v_q"], y["v_mu"], **kw)
    want = call(x)
    y = {k: a.clone() for k, a in x.items()}
    out = {"g_q": y[g_q] if g_q in y else torch.empty(N, device=dev()),
           "g_mu": y[g_mu] if g_mu else torch.empty(N, 3, device=dev())}
    if g_q == "shifted":   # begins inside the dipole tangent
        room = torch.empty(4 * N, device=dev())
        room[:3 * N] = y["v_mu"].reshape(-1)
        y["v_mu"], out["g_q"] = room[:3 * N].view(N, 3), room[2 * N:3 * N]
    got = call(y, out=out)
    for k in ("g_q", "g_mu"):
        assert rms_rel(host(got[k]), host(want[k])) <= TOL, k


@pytest.mark.parametrize("place", [{"dU_dmu": "mu"}, {"dU_dpos": "pos", "dU_dq": "q", "dU_dmu": "mu"},
                                   {"dU_dq": "pol"}, {"dU_dpos": "mu"}])
def test_model(place):
    from paper_2606_01598_amd import _lib
    plan, pme, box, x = _setup()
    want = plan.model(pme, x["pos"], x["q"], x["mu"], x["pol"], box, dU_dq=True)
    y = {k: a.clone() for k, a in x.items()}
    out = {k: y[place[k]] if k in place else torch.empty_like(a) for k, a in want.items()}
    p = lambda a: a.data_ptr()   # noqa: E731
    _lib.check(_lib.load().pol_model(plan.handle, pme.handle, torch.cuda.current_stream().cuda_stream, N,
                                     p(y["pos"]), p(y["q"]), p(y["mu"]), p(y["pol"]), p(box),
                                     p(out["energy"]), p(out["dU_dpos"]), p(out["dU_dq"]),
                                     p(out["dU_dmu"])))
    for k, a in want.items():
        assert rms_rel(host(out[k]), host(a)) <= TOL, k
