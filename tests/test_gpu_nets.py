"""Edges of the matrix-core network kernels (16 atoms a tile, 256 tiles a round of the
parameter gradients) against the FP64 oracle: one atom, tiles that are one short, full
and one over, a second round, and parameters that start off a 16-byte boundary.

Tolerance: the longest chain is three contractions of 64 (and 16 atoms per step of a
parameter gradient, up to 4097 in all): rounding of 2^-24 a step, summed as the square
root, is below 1e-5 of the RMS.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev, f32, host, rms_rel
from oracle import dip as odip, heads as oheads

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4097])
def test_network_kernels(n):
    from paper_2606_01598_amd.dip import DipPlan
    rng = np.random.default_rng(n)
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=dev())   # noqa: E731
    off = lambda a: torch.cat([torch.zeros(1, device=dev()), t(a)])[1:]   # noqa: E731
    x, xd = rng.normal(0, 1, (n, 34)), rng.normal(0, 1, (n, 34))
    V, Vd = rng.normal(0, 1, (n, 16, 3)), rng.normal(0, 1, (n, 16, 3))
    g = [rng.normal(0, 1, (n, 3)) for _ in range(4)]
    gq = [rng.normal(0, 1, n) for _ in range(3)]
    z = rng.normal(0, 1, n)
    th = f32(synth.mlp_init(3, last_scale=1.0) + rng.normal(0, 0.05, 7440))
    thq = f32(synth.charge_head_init(4, last_scale=1.0, bias_scale=0.3))
    plan = DipPlan(np.eye(3) * 30.0, n, cutoff=5.0)
    P, Q = off(th), off(thq)
    r = lambda *a: [f32(v) for v in a]   # noqa: E731
    (x, xd, V, Vd, z), g, gq = r(x, xd, V, Vd, z), r(*g), r(*gq)
    mu, mud, w, wd, cache = oheads.dipoles_jvp(th, x, V, xd, Vd)
    errs = {"mu": (plan.forward(P, t(x), t(V)), mu)}
    m, md = plan.forward_jvp(P, t(x), t(V), t(xd), t(Vd))
    errs["mu_jvp"], errs["mu_dot"] = (m, mu), (md, mud)
    gs = g[0] + g[1] + g[2]
    errs["backward"] = (plan.backward(P, t(x), t(V), *map(t, g[:3])),
                        odip.mlp_backward(th, odip.mlp(th, x)[1], np.einsum("nd,ncd->nc", gs, V)))
    gw = np.einsum("nd,ncd->nc", g[0] + g[1], V) + np.einsum("nd,ncd->nc", g[3], Vd)
    a, b = plan.backward_jvp(P, Q, t(x), t(V), t(xd), t(Vd), t(g[0]), t(g[1]), t(g[3]), t(gq[0]),
                             t(gq[1]), t(gq[2]))
    errs["backward_jvp"] = (a, oheads.mlp_jvp_backward(th, cache, gw, np.einsum("nd,ncd->nc", g[3], V)))
    c, cd, qc = oheads.charge_jvp(thq, x, xd)
    q, qd = plan.charges(Q, t(z), t(x), t(xd), q_dot=True)
    scale = float(np.sqrt(np.mean(c * c) + np.mean(cd * cd)))   # a lone atom's centred c is zero
    errs["q_backward"] = (b, oheads.charge_jvp_backward(thq, qc, oheads.centre(gq[0] + gq[1]),
                                                        oheads.centre(gq[2])))
    out = {k: rms_rel(host(u), v, 1e-3) for k, (u, v) in errs.items()}
    out["q"] = float(np.abs(host(q) - z - oheads.centre(c)).max() / scale)
    out["q_dot"] = float(np.abs(host(qd) - oheads.centre(cd)).max() / scale)
    print(n, {k: f"{v:.1e}" for k, v in out.items()}, flush=True)
    assert max(out.values()) <= TOL, out
