"""The optimal influence function's tables on pencil meshes: made, taken again and made anew
as the cell changes, each evaluation equals a fresh plan's bit for bit, through transforms in
two stages and in more, with odd and even axes and a last kz block of one to five values."""
import numpy as np
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh", [(12, 160, 150), (5, 160, 160), (125, 144, 144), (15, 243, 108)],
                         ids=lambda m: "x".join(map(str, m)))
def test_tables_follow_the_cell(mesh):
    from paper_2606_01598_amd.pme import Plan
    rng = np.random.default_rng(sum(mesh))
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=dev())   # noqa: E731
    n = 200
    s, q, mu = rng.uniform(0, 1, (n, 3)), t(rng.normal(0, 1, n)), t(rng.normal(0, 0.2, (n, 3)))
    v = [t(rng.normal(0, 1, x)) for x in ((n, 3), (n,), (n, 3))]
    cells = []
    for k in range(2):
        c = np.diag([(0.9 + 0.01 * k) * m for m in mesh])
        c[1, 0] = 0.1 * c[0, 0]
        cells.append((t(s @ c), torch.tensor(c, device=dev())))

    def both(plan, k):
        pos, box = cells[k]
        return {**plan.forward(pos, q, mu, box), **plan.backward(pos, q, mu, box, *v)}
    make = lambda: Plan(mesh, 4, 0.35, max_atoms=n, optimal_influence=True)   # noqa: E731
    fresh = [both(make(), k) for k in range(2)]
    plan = make()
    for k in (0, 0, 1, 1, 0, 1):
        out = both(plan, k)
        plan.status()
        for name, x in out.items():
            assert torch.equal(x, fresh[k][name]), (k, name)
