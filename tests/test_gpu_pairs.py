"""Edges of the wavefront-per-atom pair and feature kernels and of the cell list they
read, against the FP64 oracle: one to four cells along an axis (and mixed), atoms with no
neighbour and with more than the 128 pairs a wavefront queues, positions outside the
cell, and both cell sorts (one workgroup, or four launches).

Tolerance: a displacement carries the rounding of its positions and of the shift, at
most 2^-24 of the cell's width (3e-6 of the closest pair), which the steepest screened
function takes to the seventh power; 64 pair terms add their own 1e-6.  5e-5 covers it.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_util import RMS_REL_TOL, dev, f32, host, rms_rel
from oracle import dip as odip, heads as oheads, pol as opol

pytestmark = pytest.mark.gpu
TOL = 5e-5

# n, cell edges, cutoff, share of the atoms drawn into a cluster
CASES = {
    "two_atoms": (2, (13.0, 14.0, 15.0), 6.0, 1.0),
    "two_cells": (65, (13.0, 13.0, 13.0), 6.4, 0.0),
    "mixed_cells": (257, (13.0, 20.0, 26.5), 6.4, 0.0),
    "four_cells": (701, (27.0, 27.0, 27.0), 6.5, 0.0),
    "crowded": (420, (30.0, 30.0, 30.0), 7.0, 0.8),
    "four_launch_sort": (600, (75.0, 75.0, 75.0), 3.0, 0.9),
}


def _case(name):
    n, edges, rc, crowd = CASES[name]
    rng = np.random.default_rng(len(name))
    box = np.diag(edges)
    box[1, 0], box[2, 1] = 0.08 * edges[0], -0.05 * edges[1]
    # points kept 1.1 Angstrom apart, part of them within a small ball across a corner
    pos = np.zeros((0, 3))
    while len(pos) < n:
        frac = rng.uniform(-0.5, 0.5, 3)
        if len(pos) < crowd * n:
            frac *= 1.6 * n ** (1 / 3) / np.array(edges)
        r = frac @ box
        d = (pos - r) @ np.linalg.inv(box)
        d = (d - np.round(d)) @ box
        if not len(pos) or (d * d).sum(1).min() > 1.21:
            pos = np.vstack([pos, r])
    shift = rng.integers(-1, 2, (n, 3)) @ box   # any periodic image
    pos = pos + shift
    q = rng.normal(0, 1, n)
    # the oracle searches the images next to the cell: it takes the library's float32
    # positions moved back by the same lattice vectors
    return box, rc, pos, shift, q, rng.normal(0, 0.3, (n, 3)), rng.uniform(0.2, 3.0, n), rng


@pytest.mark.parametrize("name", CASES)
def test_pair_kernels(name):
    from paper_2606_01598_amd.pol import PolPlan
    box, rc, pos, shift, q, mu, pol, rng = _case(name)
    alpha, n = 0.35, len(q)
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=dev())   # noqa: E731
    v = rng.normal(0, 1, (n, 3))
    plan = PolPlan(box, alpha, rc, max_atoms=n)
    x = [f32(pos) - shift, f32(q), f32(mu)]
    out = plan.real(t(pos), t(q), t(mu), t(pol), dE_dq=True)
    e, gp, gm = opol.real_space(*x, box, alpha, rc, f32(pol))
    gq = opol.real_charge_grad(*x, box, alpha, rc, f32(pol))
    mixed = plan.mixed(t(pos), t(q), t(mu), t(pol), t(v))
    ref = opol.real_mixed(*x, box, alpha, rc, f32(pol), f32(v))
    errs = {"E": abs(float(host(out["energy"])[0]) - e) / np.abs(x[1] * gq).sum() if e else 0.0,
            "dE_dpos": rms_rel(host(out["dE_dpos"]), gp), "dE_dq": rms_rel(host(out["dE_dq"]), gq),
            "dE_dmu": rms_rel(host(out["dE_dmu"]), gm), "mixed": rms_rel(host(mixed), ref)}
    print(name, {k: f"{w:.2e}" for k, w in errs.items()}, flush=True)
    assert max(errs.values()) <= TOL, errs


@pytest.mark.parametrize("name", CASES)
def test_feature_kernels(name):
    from paper_2606_01598_amd.dip import DipPlan
    box, rc, pos, shift, q, _, _, rng = _case(name)
    n = len(q)
    t = lambda a: torch.tensor(a, dtype=torch.float32, device=dev())   # noqa: E731
    v, u = rng.normal(0, 1, (n, 3)), rng.normal(0, 1, (n, 3))
    theta = f32(synth.mlp_init(5, last_scale=1.0))
    plan = DipPlan(box, n, cutoff=rc)
    feat, vec = plan.features(t(pos), t(q))
    fd, vd = plan.features_jvp(t(pos), t(q), vec, t(v))
    base = rng.normal(0, 1, (n, 3))
    g = plan.position_vjp(t(theta), t(pos), t(q), feat, vec, t(u), base=t(base))
    x = f32(pos) - shift
    rf, rv = odip.features(x, f32(q), box, rc)
    rfd, rvd = oheads.features_jvp(x, f32(q), box, rc, f32(v))
    rg = odip.position_vjp(theta, x, f32(q), box, rc, f32(u))
    errs = {"feat": rms_rel(host(feat), rf), "vec": rms_rel(host(vec), rv),
            "feat_dot": rms_rel(host(fd), rfd), "vec_dot": rms_rel(host(vd), rvd)}
    eg = rms_rel(host(g) - f32(base), rg)
    print(name, {k: f"{w:.2e}" for k, w in errs.items()}, f"vjp {eg:.2e}", flush=True)
    assert max(errs.values()) <= TOL, errs
    assert eg <= RMS_REL_TOL
