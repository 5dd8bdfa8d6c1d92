"""The pencil passes (meshes whose y-z plane exceeds LDS) at the edges of their line
groups and kz blocks: lengths in two stages and not, on each axis, 1 to 8 values in the
last kz block, odd plane counts, and fewer planes than a workgroup takes.

The potential is compared with K rho of the plan's own density in 64-bit torch.fft; its
tolerance is that of the repository's potential test (1e-5 of the RMS: some twenty
roundings of 2^-24 a value).  The cell gradient and the optimal influence function run
the other variants of the x pass, compared with the oracle to their bars.
"""
import math

import numpy as np
import pytest
import torch

import synth
from gpu_util import E_REL_TOL, RMS_REL_TOL, dev, f32, host, rel, rms_rel
from oracle import pme as opme

pytestmark = pytest.mark.gpu

# two stages unless named: x 5 and 125, y 250 and 243, z 125 and 250
MESHES = [(12, 160, 150), (16, 144, 162), (5, 160, 160), (125, 144, 144), (9, 250, 128),
          (15, 243, 108), (10, 162, 125), (6, 128, 250), (27, 160, 135), (8, 320, 324)]


def _frame(n, mesh, seed):
    rng = np.random.default_rng(seed)
    box = np.diag([0.9 * m for m in mesh])
    box[1, 0] = 0.1 * box[0, 0]
    q = rng.normal(0, 1, n)
    return synth.Frame(pos=rng.uniform(0, 1, (n, 3)) @ box, q=q - q.mean(),
                       mu=rng.normal(0, 0.2, (n, 3)), box=box)


def _args(f):
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=dev())   # noqa: E731
    return t(f.pos), t(f.q), t(f.mu), torch.tensor(f.box, device=dev())


@pytest.mark.parametrize("mesh", MESHES, ids=lambda m: "x".join(map(str, m)))
def test_potential_matches_fft(mesh):
    from paper_2606_01598_amd.pme import Plan
    p, alpha = 4, 0.35
    f = _frame(300, mesh, sum(mesh))
    plan = Plan(mesh, p, alpha, max_atoms=f.n)
    x = _args(f)
    out = plan.forward(*x)
    plan.status()
    rho, phi = plan.rho().double(), plan.phi().double()
    fr = [torch.fft.fftfreq(m, 1.0 / m, dtype=torch.float64, device=dev()) for m in mesh]
    k = torch.stack(torch.meshgrid(*fr, indexing="ij"), -1) @ (2 * math.pi * torch.linalg.inv(x[3]).T)
    k2 = (k * k).sum(-1)
    k2[0, 0, 0] = 1.0
    g = 4 * math.pi / k2 * torch.exp(-k2 / (4 * alpha ** 2))
    g[0, 0, 0] = 0.0
    for a in range(3):
        shape = [1, 1, 1]
        shape[a] = mesh[a]
        g = g * (torch.sinc(fr[a] / mesh[a]) ** (-2 * p)).reshape(shape)
    ref = torch.fft.ifftn(g * torch.fft.fftn(rho)).real * rho.numel()
    err = rms_rel(host(phi), host(ref))
    e = float((rho * ref).sum() / (2 * torch.linalg.det(x[3]).abs()))
    print(mesh, f"{err:.2e} {rel(host(out['energy'])[0], e):.2e}", flush=True)
    assert err <= 1e-5 and rel(host(out["energy"])[0], e) <= E_REL_TOL


@pytest.mark.parametrize("mesh", [(5, 160, 150), (12, 160, 150)], ids=["general_x", "two_stage_x"])
def test_cell_gradient_and_optimal_influence(mesh):
    from paper_2606_01598_amd.pme import Plan
    p, alpha = 4, 0.35
    f = _frame(40, mesh, 3)
    x = _args(f)
    ref = (f32(f.pos), f32(f.q), f32(f.mu), f.box, mesh, p, alpha)
    out = Plan(mesh, p, alpha, max_atoms=f.n).forward(*x, cell=True)
    cell = opme.cell_gradient(*ref)
    err = np.abs(host(out["dE_dbox"]) - cell).max() / np.abs(cell).max()
    plan = Plan(mesh, p, alpha, max_atoms=f.n, optimal_influence=True)
    best = opme.forward(*ref, gamma="optimal")
    errs = []
    for _ in range(2):   # the tables made, then taken
        o = plan.forward(*x)
        errs += [rms_rel(host(o[k]), getattr(best, k)) for k in ("dE_dpos", "dE_dq", "dE_dmu")]
        errs.append(rel(host(o["energy"])[0], best.e_recip) * RMS_REL_TOL / E_REL_TOL)
    print(mesh, f"cell {err:.1e} optimal {max(errs):.1e}", flush=True)
    assert err <= 2e-5 and max(errs) <= RMS_REL_TOL
