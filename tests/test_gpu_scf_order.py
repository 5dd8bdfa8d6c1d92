"""pol_scf returns when its work is done: the stream has nothing left to run, so that another
stream or thread may read the dipoles at once."""
import numpy as np
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,max_iter", [(60, 40), (4000, 40), (4000, 3), (4000, 0)])
def test_nothing_in_flight_after_a_solve(n, max_iter):
    from paper_2606_01598_amd.pme import Plan
    from paper_2606_01598_amd.pol import PolPlan
    rng = np.random.default_rng(n)
    k = int(np.ceil(n ** (1 / 3)))
    side = max(13.0, 3.15 * k)
    at = np.stack(np.unravel_index(rng.permutation(k ** 3)[:n], (k, k, k)), 1)
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=dev())   # noqa: E731
    pos, q = t((at + rng.uniform(-0.1, 0.1, (n, 3))) * side / k), t(np.where(np.arange(n) % 2, 1.0, -1.0))
    pol, box = t(rng.uniform(0.2, 2.0, n)), torch.tensor(np.eye(3) * side, device=dev())
    pme = Plan((48,) * 3, 6, 0.3, max_atoms=n)
    plan = PolPlan(box, 0.3, 6.0, max_atoms=n)
    mu = torch.zeros(n, 3, device=dev())
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        idle = []
        for _ in range(20):
            plan.scf(pme, pos, q, pol, box, tol=1e-6, max_iter=max_iter, mu=mu)
            idle.append(stream.query())
    torch.cuda.synchronize()
    assert all(idle), idle
