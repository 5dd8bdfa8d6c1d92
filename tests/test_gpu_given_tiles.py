"""Plans with given tiles whose edges do not divide the mesh, where a tile holds many atom
bins: every atom gets its outputs (the buffers hold NaN before each call), which agree with
the FP64 oracle to the bars of the other parity tests.  Axes of threes, on which the tuner's
16 x 16 x 16 target becomes 15; tiles long in z and in x; a mesh spread by bands; and the
same meshes in a batch."""
import pytest
import torch

import synth
from gpu_util import E_REL_TOL, RMS_REL_TOL, host, oracle_forward, oracle_hvp, rel, rms_rel, to_dev

pytestmark = pytest.mark.gpu

CASES = {"cube27": ((27, 27, 27), (16, 16, 16), "fused"), "cube54": ((54, 54, 54), (16, 16, 16), "fused"),
         "mixed": ((54, 60, 54), (16, 16, 16), "fused"), "long_z": ((27, 27, 81), (8, 8, 32), "fused"),
         "long_x": ((40, 40, 40), (32, 12, 12), "fused"),
         "band": ((27, 162, 162), (16, 16, 16), "band")}


def _nan(shapes, device):
    return {k: torch.full(s, float("nan"), dtype=torch.float64 if k == "energy" else torch.float32,
                          device=device) for k, s in shapes.items()}


def _frame(n, mesh, seed):
    import numpy as np
    rng = np.random.default_rng(seed)
    box = np.diag([0.8 * m for m in mesh])
    q = rng.normal(0.0, 1.0, n)
    return synth.Frame(pos=rng.uniform(0.0, 1.0, (n, 3)) @ box, q=q - q.mean(),
                       mu=rng.normal(0.0, 0.1, (n, 3)), box=box)


@pytest.mark.parametrize("case", CASES)
def test_every_atom_of_a_given_tile(case):
    from paper_2606_01598_amd.pme import Plan
    mesh, tile, spread = CASES[case]
    p, alpha, n = 4, 0.4, 900
    print(f"case: {case} mesh={mesh} tile={tile}", flush=True)
    f = _frame(n, mesh, sum(mesh))
    v = synth.random_cotangents(n, 7, scale_r=0.1)
    ref = oracle_forward(f, mesh, p, alpha, 1.0, with_q=True, with_mu=True)
    href = oracle_hvp(f, mesh, p, alpha, v)
    want = {"dE_dpos": ref.dE_dpos, "dE_dq": ref.dE_dq, "dE_dmu": ref.dE_dmu,
            "g_pos": href[0], "g_q": href[1], "g_mu": href[2]}
    args = to_dev(f)
    d = args[0].device
    vd = [torch.tensor(x, dtype=torch.float32, device=d) for x in v]
    fwd = {"energy": (3,), "dE_dpos": (n, 3), "dE_dq": (n,), "dE_dmu": (n, 3)}
    bwd = {"g_pos": (n, 3), "g_q": (n,), "g_mu": (n, 3)}
    plan = Plan(mesh, p, alpha, max_atoms=n, tile=tile)
    both = Plan(mesh, p, alpha, max_atoms=n, tile=tile, concurrent=True)
    assert plan.spread_kind == spread
    apart = {**plan.forward(*args, out=_nan(fwd, d)), **plan.backward(*args, *vd, out=_nan(bwd, d))}
    step = both.step(*args, *vd, out=_nan({**fwd, **bwd}, d))
    plan.status()
    both.status()
    for name, out in (("apart", apart), ("step", step)):
        assert rel(host(out["energy"]).sum(), ref.energy) <= E_REL_TOL, name
        for k, w in want.items():
            assert rms_rel(host(out[k]), w) <= RMS_REL_TOL, (name, k)


def test_batch_of_given_tiles():
    from paper_2606_01598_amd.batch import Batch
    p, alpha = 4, 0.4
    cases = [CASES[k] for k in ("cube27", "cube54", "long_z")]
    frames = [_frame(500 + 100 * b, m, b) for b, (m, _, _) in enumerate(cases)]
    bt = Batch([c[0] for c in cases], [f.n for f in frames], p, alpha, tiles=[c[1] for c in cases])
    parts = [to_dev(f) for f in frames]
    pos, q, mu = (torch.cat([t[k] for t in parts]) for k in range(3))
    box = torch.stack([t[3] for t in parts])
    v = [synth.random_cotangents(f.n, 3, scale_r=0.1) for f in frames]
    vd = [torch.cat([torch.tensor(t[k], dtype=torch.float32, device=pos.device) for t in v])
          for k in range(3)]
    fo, bo = bt.forward(pos, q, mu, box), bt.backward(pos, q, mu, box, *vd)
    o = 0
    for b, f in enumerate(frames):
        s = slice(o, o + f.n)
        o += f.n
        ref = oracle_forward(f, cases[b][0], p, alpha, 1.0, with_q=True, with_mu=True)
        href = oracle_hvp(f, cases[b][0], p, alpha, v[b])
        for k in ("dE_dpos", "dE_dq", "dE_dmu"):
            assert rms_rel(host(fo[k][s]), getattr(ref, k)) <= RMS_REL_TOL, (b, k)
        for k, w in zip(("g_pos", "g_q", "g_mu"), href):
            assert rms_rel(host(bo[k][s]), w) <= RMS_REL_TOL, (b, k)
