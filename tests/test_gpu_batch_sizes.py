"""Batches at the edges of their dispatch: every box equals a plan of its own bit for
bit.  Planes of 4096 points (the most that go in small workgroups, with the spread fused)
and one box beyond; a mesh too small for a plane spread; long planes of few rows, whose
fused workspace exceeds a small workgroup's, or does with its static LDS; x lines of 128 points and beyond; one row of
butterflies more than a small workgroup; a box with more atoms in a plane than are
listed at a time."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

CASES = {"most": [(64, 64, 64), (16, 16, 16)], "beyond": [(20, 80, 64), (16, 16, 16)],
         "tiny": [(8, 8, 8), (16, 18, 20)], "long": [(16, 10, 400), (16, 16, 16)],
         "brim": [(12, 9, 450), (12, 9, 405)],
         "lines": [(128, 16, 20), (18, 16, 16)], "more_lines": [(135, 16, 20), (18, 16, 16)],
         "odd": [(45, 27, 25), (30, 36, 45), (50, 20, 50)], "crowded": [(12, 45, 48)]}


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("p", [4, 6])
def test_batch_equals_plans(case, p):
    from paper_2606_01598_amd.batch import Batch
    from paper_2606_01598_amd.pme import Plan
    meshes = CASES[case]
    print(f"case: {case} p={p}", flush=True)
    counts = [3000 if case == "crowded" else 60 + 30 * b for b in range(len(meshes))]
    frames = []
    for b, n in enumerate(counts):
        rng = np.random.default_rng(70 + b)
        frames.append(synth.Frame(pos=rng.uniform(0.0, 22.0, (n, 3)), q=rng.normal(0.0, 1.0, n),
                                  mu=rng.normal(0.0, 0.1, (n, 3)), box=22.0 * np.eye(3)))
    bt = Batch(meshes, counts, p, 0.4)
    parts = [to_dev(f) for f in frames]
    pos, q, mu = (torch.cat([t[k] for t in parts]) for k in range(3))
    box = torch.stack([t[3] for t in parts])
    g = torch.Generator().manual_seed(3)
    v = [torch.randn(x.shape, generator=g).to(x) for x in (pos, q, mu)]
    fo = bt.forward(pos, q, mu, box)
    bo = bt.backward(pos, q, mu, box, *v)
    o = 0
    for b, n in enumerate(counts):
        plan = Plan(meshes[b], p, 0.4, max_atoms=n)
        s = slice(o, o + n)
        o += n
        f1 = plan.forward(*parts[b])
        b1 = plan.backward(*parts[b], *(x[s].contiguous() for x in v))
        plan.status()
        assert torch.equal(fo["energy"][b], f1["energy"]), b
        for k in ("dE_dpos", "dE_dq", "dE_dmu"):
            assert torch.equal(fo[k][s], f1[k]), (b, k)
        for k in ("g_pos", "g_q", "g_mu"):
            assert torch.equal(bo[k][s], b1[k]), (b, k)
