"""The quadrupole forward and the batches that spread tiles read cubic atom bins, in the
counters and records that the plan's other calls use with bins one cell wide: calls of both
kinds in any order on one plan give what fresh plans give, bit for bit (meshes with more
bins of either kind, and one spread by bands)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh,spread", [((27, 32, 32), "fused"), ((30, 40, 40), "fused"),
                                         ((20, 135, 128), "band")])
@pytest.mark.parametrize("concurrent", [False, True])
def test_calls_of_both_views_in_any_order(mesh, spread, concurrent):
    from paper_2606_01598_amd.pme import Plan
    n, p, alpha = 900, 6, 0.35
    rng = np.random.default_rng(sum(mesh))
    box = np.diag([0.9 * m for m in mesh])
    # a third of the atoms in one corner: bins of both kinds pass their capacity
    pos = rng.uniform(0, 1, (n, 3)) @ box
    pos[::3] *= 0.2
    f = synth.Frame(pos=pos, q=rng.normal(0, 1, n), mu=rng.normal(0, 0.1, (n, 3)), box=box)
    args = to_dev(f)
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=args[0].device)   # noqa: E731
    theta, v = t(rng.normal(0, 0.2, (n, 6))), [t(x) for x in synth.random_cotangents(n, 5)]
    calls = {"f": lambda pl: pl.forward(*args), "q": lambda pl: pl.forward(*args, theta=theta),
             "b": lambda pl: pl.backward(*args, *v), "s": lambda pl: pl.step(*args, *v)}
    make = lambda: Plan(mesh, p, alpha, max_atoms=n, concurrent=concurrent)   # noqa: E731
    fresh = {}
    for k, call in calls.items():
        plan = make()
        assert plan.spread_kind == spread
        fresh[k] = call(plan)
        plan.status()
    plan = make()
    for i, k in enumerate("qfqqbfbqsqssqfsq"):
        out = calls[k](plan)
        for name, x in out.items():
            assert torch.equal(x, fresh[k][name]), (i, k, name)
    plan.status()
