"""Timed workloads of the library: what a simulation, a training run and the teacher
that labels it call, each through the public Python entry points.

``listed()`` names the standing cases and ``draw(rng)`` makes more of the same ranges.
``prepare`` builds what a program holds before the call (plan, inputs, buffers),
``run`` is one pass, ``work`` its least bytes and operations, and ``exact`` the same
outputs from plain 64-bit torch.

Inputs are molten-salt-like: ions at 1000 per (31.5 Angstrom)^3 on jittered lattice
sites (closest pairs about 2.2 Angstrom) in random order, charges +-1 that mostly
alternate between neighbours, dipoles of 0.1 e Angstrom, meshes near one point per
Angstrom.  Energies and cell gradients are returned in the type of the forces, as a
training loss takes them.
"""
import math
import random

import numpy as np
import torch

from paper_2606_01598_amd.batch import Batch
from paper_2606_01598_amd.dip import NPARAM, NQPARAM, DipPlan, Trainer
from paper_2606_01598_amd.pme import Plan, pme_energy
from paper_2606_01598_amd.pol import PolPlan, teacher

DENSITY = 1000.0 / 31.5 ** 3
POL_CATION, POL_ANION = 0.15, 3.5   # polarizabilities of the Thole boxes, Angstrom^3
R_PAIR, R_FEAT = 10.0, 5.0          # real-space and feature cutoffs, Angstrom
SMOOTH = sorted({2 ** a * 3 ** b * 5 ** c for a in range(10) for b in range(6) for c in range(4)
                 if 16 <= 2 ** a * 3 ** b * 5 ** c <= 320})
PME_KINDS = ("energy", "forward", "force_loss", "step", "replay", "stress")


def listed():
    def pme(name, kind, atoms, mesh, order=6, alpha=0.30, tilt=0.0):
        return {"name": name, "kind": kind, "atoms": atoms, "mx": mesh[0], "my": mesh[1],
                "mz": mesh[2], "order": order, "alpha": alpha, "tilt": tilt}

    def thole(name, kind, atoms, mesh):
        return {"name": name, "kind": kind, "atoms": atoms, "mx": mesh, "my": mesh, "mz": mesh,
                "order": 6, "alpha": 0.30, "tilt": 0.0}

    return [
        # the smallest call: energy and gradients of one small cell through autograd
        pme("energy_64", "energy", 64, (16, 16, 16), order=4),
        # energy and forces of a small simulation box, plan kept between steps
        pme("forward_1k", "forward", 1000, (32, 32, 32)),
        # a force loss through autograd with create_graph, on an odd-sized box
        pme("force_loss_5k", "force_loss", 5402, (60, 50, 54), order=5, alpha=0.35),
        # a training step's forward and Hessian-vector product, two steps per captured graph
        pme("replay_8k", "replay", 8000, (64, 64, 64)),
        # the benchmark's step, as eager calls
        pme("step_32k", "step", 32000, (100, 100, 100)),
        # the same on a mesh whose planes exceed LDS
        pme("step_128k", "step", 128000, (160, 160, 160)),
        # the largest box of the size sweep
        pme("step_1m", "step", 1000000, (320, 320, 320)),
        # energy, forces and cell gradient of a sheared box (variable-cell simulation)
        pme("stress_21k", "stress", 21390, (90, 81, 96), order=5, tilt=0.13),
        # one training step of Eq. loss over a batch of small boxes, as a captured graph
        {"name": "batch_64", "kind": "batch", "boxes": 64, "layout": 6, "least": 64,
         "most": 4096, "order": 6, "alpha": 0.30},
        # labelling one box with the self-consistent polarizable teacher
        thole("teacher_4096", "teacher", 4096, 50),
        # simulation with the learned heads: features, charges, dipoles, conservative forces
        thole("student_4096", "student", 4096, 50),
        # one training step of both learned heads on conservative forces
        thole("train_4096", "train", 4096, 50),
    ]


def draw(rng):
    def log_int(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(PME_KINDS + ("step", "batch", "teacher", "student", "train"))
    if kind == "batch":
        return {"kind": kind, "boxes": log_int(6, 64), "layout": rng.randrange(1 << 20),
                "least": 64, "most": log_int(600, 4096), "order": rng.choice((5, 6)),
                "alpha": 0.30}
    if kind in ("teacher", "student", "train"):
        atoms = 2 * log_int(300, 2048)
        side = _near_smooth((atoms / DENSITY) ** (1 / 3))
        return {"kind": kind, "atoms": atoms, "mx": side, "my": side, "mz": side, "order": 6,
                "alpha": 0.30, "tilt": 0.0}
    most = {"energy": 16000, "forward": 60000, "force_loss": 40000, "replay": 64000,
            "step": 1000000, "stress": 100000}[kind]
    atoms = 2 * log_int(32 if kind == "energy" else 400, most / 2)
    side = (atoms / DENSITY) ** (1 / 3) * rng.uniform(0.85, 1.05)
    a, b = rng.uniform(0.85, 1.18), rng.uniform(0.85, 1.18)
    mesh = [_near_smooth(side * f) for f in (a, b, 1 / (a * b))]
    while mesh[0] * mesh[1] * mesh[2] > 320 ** 3:
        k = mesh.index(max(mesh))
        mesh[k] = SMOOTH[SMOOTH.index(mesh[k]) - 1]
    return {"kind": kind, "atoms": atoms, "mx": mesh[0], "my": mesh[1], "mz": mesh[2],
            "order": rng.choice((4, 5, 6, 6)), "alpha": rng.choice((0.30, 0.35)),
            "tilt": round(rng.uniform(0.02, 0.2), 3) if kind == "stress" or rng.random() < 0.2 else 0.0}


def _near_smooth(x):
    return min(SMOOTH, key=lambda m: (abs(m - x), m))


def _batch_counts(case):
    rng = random.Random(case["layout"])
    lo, hi = math.log(case["least"] / 2), math.log(case["most"] / 2)
    return [2 * int(round(math.exp(rng.uniform(lo, hi)))) for _ in range(case["boxes"])]


def _batch_mesh(n):
    return (min(_near_smooth((n / DENSITY) ** (1 / 3)), 64),) * 3


# ---- inputs ----------------------------------------------------------------

def _melt(n, mesh, tilt, rng):
    """Positions, charges, dipoles (float32) and the cell (float64), on the host."""
    h = (n / DENSITY / (mesh[0] * mesh[1] * mesh[2])) ** (1 / 3)
    box = np.diag([m * h for m in mesh])
    box[1, 0], box[2, 0], box[2, 1] = tilt * box[0, 0], -0.7 * tilt * box[0, 0], 0.5 * tilt * box[1, 1]
    site = DENSITY ** (-1 / 3)
    k = np.array([max(1, math.ceil(box[a, a] / site - 1e-9)) for a in range(3)])
    at = np.stack(np.unravel_index(rng.permutation(int(k.prod()))[:n], k), axis=1)
    frac = (at + 0.5 + rng.uniform(-0.14, 0.14, (n, 3))) / k
    # alternating charges, evened out, then a tenth of the ions trade theirs
    q = 1.0 - 2.0 * (at.sum(axis=1) % 2)
    major = np.flatnonzero(q == np.sign(q.sum()))
    q[rng.permutation(major)[:int(abs(q.sum())) // 2]] *= -1.0
    trade = rng.permutation(n)[:n // 10]
    q[trade] = q[rng.permutation(trade)]
    return frac @ box, q, rng.normal(0.0, 0.1, (n, 3)), box


def _gpu(a):
    return torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")


def _inputs(case, seed):
    """The case's arrays as the library takes them, from the seed alone."""
    rng = np.random.default_rng(seed)
    if case["kind"] == "batch":
        parts = [_melt(n, _batch_mesh(n), 0.0, rng) for n in _batch_counts(case)]
        total = sum(len(p[1]) for p in parts)
        s = {k: _gpu(np.concatenate([p[j] for p in parts])) for j, k in enumerate(("pos", "q", "mu"))}
        s["box"] = torch.tensor(np.stack([p[3] for p in parts]), device="cuda")
        s.update(v_pos=_gpu(rng.normal(0, 0.1, (total, 3))), v_q=_gpu(rng.normal(0, 1, total)),
                 v_mu=_gpu(rng.normal(0, 1, (total, 3))), vf_pos=_gpu(rng.normal(0, 0.1, (total, 3))))
        return s
    n = case["atoms"]
    pos, q, mu, box = _melt(n, (case["mx"], case["my"], case["mz"]), case["tilt"], rng)
    s = {"pos": _gpu(pos), "q": _gpu(q), "mu": _gpu(mu), "box": torch.tensor(box, device="cuda")}
    if case["kind"] in ("step", "replay"):
        s.update(v_pos=_gpu(rng.normal(0, 0.1, (n, 3))), v_q=_gpu(rng.normal(0, 1, n)),
                 v_mu=_gpu(rng.normal(0, 1, (n, 3))))
    if case["kind"] in ("force_loss", "train"):
        s["f_ref"] = _gpu(rng.normal(0, 0.2, (n, 3)))
        s["e_ref"] = torch.tensor([-0.28 * n], dtype=torch.float64, device="cuda")
    if case["kind"] in ("teacher", "student", "train"):
        s["pol"] = _gpu(np.where(q > 0, POL_CATION, POL_ANION))
        s["theta"], s["qtheta"] = _head_parameters(rng)
    return s


def _head_parameters(rng):
    """Glorot-uniform parameters of both heads, the output layers scaled by 0.1."""
    def layer(out, inp, scale=1.0):
        lim = scale * math.sqrt(6.0 / (out + inp))
        return rng.uniform(-lim, lim, out * inp)

    z = np.zeros
    theta = np.concatenate([layer(64, 34), z(64), layer(64, 64), z(64), layer(16, 64, 0.1), z(16)])
    qtheta = np.concatenate([layer(64, 34), z(64), layer(64, 1, 0.1)])
    assert len(theta) == NPARAM and len(qtheta) == NQPARAM
    return theta, qtheta


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, p, alpha = case["kind"], case["order"], case["alpha"]
    s["kind"] = kind
    if kind == "batch":
        counts = _batch_counts(case)
        s["batch"] = Batch([_batch_mesh(n) for n in counts], counts, p, alpha)
        n, nbox = s["batch"].total, s["batch"].nbox
        new = lambda *shape: torch.empty(*shape, dtype=torch.float32, device="cuda")  # noqa: E731
        s["step"] = {k: s[k] for k in ("pos", "q", "mu", "box", "v_pos", "v_q", "v_mu", "vf_pos")}
        s["out"] = {"energy": torch.empty(nbox, 3, dtype=torch.float64, device="cuda")}
        for stem in ("dE_dX", "g_X", "gf_X"):
            for x, cols in (("pos", (3,)), ("q", ()), ("mu", (3,))):
                s["out"][stem.replace("X", x)] = new(n, *cols)
        s["batch"].capture({**s["step"], **s["out"]})
        return s
    mesh, n = (case["mx"], case["my"], case["mz"]), case["atoms"]
    s["plan"] = Plan(mesh, p, alpha, max_atoms=n, concurrent=kind in ("step", "replay"))
    if kind in ("forward", "stress", "step"):
        s["out"] = {"energy": torch.empty(3, dtype=torch.float64, device="cuda")}
        for k in ("dE_dpos", "dE_dmu") + (("g_pos", "g_mu") if kind == "step" else ()):
            s["out"][k] = torch.empty(n, 3, dtype=torch.float32, device="cuda")
        for k in ("dE_dq",) + (("g_q",) if kind == "step" else ()):
            s["out"][k] = torch.empty(n, dtype=torch.float32, device="cuda")
    if kind == "replay":
        s["out"] = s["plan"].step_capture(2, s["pos"], s["q"], s["mu"], s["box"], s["v_pos"],
                                          s["v_q"], s["v_mu"])
    if kind in ("teacher", "student", "train"):
        s["pols"] = PolPlan(s["box"], alpha, R_PAIR, max_atoms=n)
    if kind in ("student", "train"):
        s["dip"] = DipPlan(s["box"], n, cutoff=R_FEAT)
        s["trainer"] = Trainer(s["dip"], s["pols"], s["plan"], s["box"], s["theta"], lr=3e-3,
                               warmup=150, qtheta0=s["qtheta"], conservative=True)
    if kind == "train":
        # features of a training box are made once and kept with its labels
        feat, vec = s["dip"].features(s["pos"], s["q"])
        s["labelled"] = {"pos": s["pos"], "q": s["q"], "pol": s["pol"], "feat": feat, "vec": vec,
                         "U": s["e_ref"], "dUdr": s["f_ref"]}
    return s


# ---- one pass ----------------------------------------------------------------

def _single(out):
    return {k: t.float() for k, t in out.items()}


def run(s):
    kind = s["kind"]
    if kind == "batch":
        s["batch"].replay()
        return _single(s["out"])
    if kind == "replay":
        s["plan"].step_replay()
        return _single(s["out"])
    x = (s["pos"], s["q"], s["mu"], s["box"])
    if kind in ("forward", "stress"):
        return _single(s["plan"].forward(*x, out=s["out"], cell=kind == "stress"))
    if kind == "step":
        return _single(s["plan"].step(*x, s["v_pos"], s["v_q"], s["v_mu"], out=s["out"]))
    if kind in ("energy", "force_loss"):
        leaves = [t.detach().requires_grad_() for t in x[:3]]
        energy = pme_energy(*leaves, s["box"], s["plan"])
        if kind == "energy":
            return [energy.float(), *torch.autograd.grad(energy, leaves)]
        (slope,) = torch.autograd.grad(energy, leaves[0], create_graph=True)
        loss = (((energy - s["e_ref"]) / len(leaves[1])).float() ** 2).sum() + \
            (slope + s["f_ref"]).square().mean()
        return [loss, slope.detach(), *torch.autograd.grad(loss, leaves)]
    # the real-space pair sums follow a cell list filled with atomics, so the last bits of
    # the energies of the polarizable model vary from run to run; the forces are returned
    if kind == "teacher":
        out = teacher(s["pols"], s["plan"], s["pos"], s["q"], s["pol"], s["box"])
        return {"mu": out["mu"], "dU_dpos": out["dU_dpos"]}
    if kind == "student":
        feat, vec = s["dip"].features(s["pos"], s["q"])
        out = s["trainer"].evaluate({"pos": s["pos"], "q": s["q"], "pol": s["pol"], "feat": feat,
                                     "vec": vec})
        return {"feat": feat, "vec": vec, **_single(out)}
    loss = s["trainer"].step(s["labelled"])
    return {"loss": loss.float(), "grad": s["trainer"].grad, "params": s["trainer"].params}


def _pme_work(n, m, p, forward, hvps):
    """Inputs once and outputs once; separable stencil sums (2 flops per FMA) and the
    real transforms (2.5 M log2 M each)."""
    fft = 5.0 * m * math.log2(m)
    evals = forward + hvps
    return {"bytes": 28.0 * n * evals + 28.0 * n * evals,
            "flops": evals * fft + n * p ** 3 * (10.0 * forward + 20.0 * hvps)}


def work(case):
    kind, p = case["kind"], case["order"]
    if kind == "batch":
        parts = [_pme_work(n, math.prod(_batch_mesh(n)), p, 1, 2) for n in _batch_counts(case)]
        return {k: sum(w[k] for w in parts) for k in ("bytes", "flops")}
    n, m = case["atoms"], case["mx"] * case["my"] * case["mz"]
    hvps = {"step": 1, "replay": 1, "force_loss": 1, "train": 1}.get(kind, 0)
    w = _pme_work(n, m, p, 1, hvps)
    if kind == "replay":
        w = {k: 2 * v for k, v in w.items()}
    pairs = n * DENSITY * 4 / 3 * math.pi * R_PAIR ** 3
    near = n * DENSITY * 4 / 3 * math.pi * R_FEAT ** 3
    if kind == "teacher":   # about eleven matrix-vector products, each a transform and a pair sum
        w["flops"] = 12 * (w["flops"] + 60.0 * pairs)
    if kind in ("student", "train"):
        nets = 2.0 * n * (NPARAM + NQPARAM)
        times = 3 if kind == "student" else 10
        w["flops"] += times * nets + (2 if kind == "train" else 1) * (100.0 * pairs + 300.0 * near)
        w["bytes"] += 4.0 * n * (34 + 48) * (1 if kind == "student" else 2)
    return w


# ---- the same outputs in 64 bits, plain torch ----------------------------------

def _splines(f, p):
    """N_p(f + p - 1 - j) and its derivative, j = 0 .. p - 1 (last axis)."""
    v = [torch.ones_like(f)]
    below = v
    for k in range(2, p + 1):
        below, prev = v, v + [torch.zeros_like(f)]
        v = [((f + i) * prev[i] + ((k - f - i) * prev[i - 1] if i else 0)) / (k - 1) for i in range(k)]
    low = below + [torch.zeros_like(f)]
    d = [low[i] - (low[i - 1] if i else 0) for i in range(p)]
    return torch.stack(v[::-1], -1), torch.stack(d[::-1], -1)


def _footprint(pos, q, mu, box, mesh, p):
    """Mesh indices and values of the density, (n, p^3) each."""
    size = torch.tensor(mesh, dtype=torch.float64, device=pos.device)
    inv = torch.linalg.inv(box)
    frac = pos @ inv
    x = (frac - torch.floor(frac)) * size + (0.5 if p & 1 else 0.0)
    cell = torch.floor(x)
    w, dw = _splines(x - cell, p)
    d = (mu @ inv) * size
    j = torch.arange(p, device=pos.device) - (p - 1) // 2
    i = [(cell[:, a, None].long() + j) % mesh[a] for a in range(3)]
    at = (i[0][:, :, None, None] * mesh[1] + i[1][:, None, :, None]) * mesh[2] + i[2][:, None, None, :]
    wx, wy, wz = w[:, 0, :, None, None], w[:, 1, None, :, None], w[:, 2, None, None, :]
    dx, dy, dz = dw[:, 0, :, None, None], dw[:, 1, None, :, None], dw[:, 2, None, None, :]
    c = [t[:, None, None, None] for t in (q, d[:, 0], d[:, 1], d[:, 2])]
    val = c[0] * wx * wy * wz + c[1] * dx * wy * wz + c[2] * wx * dy * wz + c[3] * wx * wy * dz
    return at.reshape(len(pos), -1), val.reshape(len(pos), -1)


def _convolve(rho, box, mesh, p, alpha):
    """K rho: the influence function of the assignment of order p, unnormalised inverse."""
    f = [torch.fft.fftfreq(m, 1.0 / m, dtype=torch.float64, device=rho.device) for m in mesh]
    k = torch.stack(torch.meshgrid(*f, indexing="ij"), -1) @ (2 * math.pi * torch.linalg.inv(box).T)
    k2 = (k * k).sum(-1)
    zero = torch.zeros_like(k2, dtype=torch.bool)
    zero[0, 0, 0] = True
    k2 = torch.where(zero, 1.0, k2)
    g = torch.where(zero, 0.0, 4 * math.pi / k2 * torch.exp(-k2 / (4 * alpha ** 2)))
    for a in range(3):
        shape = [1, 1, 1]
        shape[a] = mesh[a]
        g = g * (torch.sinc(f[a] / mesh[a]).abs() ** (-2 * p)).reshape(shape)
    return torch.fft.ifftn(g * torch.fft.fftn(rho.reshape(mesh))).real.reshape(-1) * rho.numel()


def _volume(box):
    return torch.linalg.det(box).abs()


def _parts_recip(pos, q, mu, box, mesh, p, alpha):
    """[E_recip, E_self_q, E_self_mu] as one differentiable expression (small boxes)."""
    at, val = _footprint(pos, q, mu, box, mesh, p)
    rho = torch.zeros(math.prod(mesh), dtype=torch.float64, device=pos.device)
    rho = rho.index_add(0, at.reshape(-1), val.reshape(-1))
    recip = (rho * _convolve(rho, box, mesh, p, alpha)).sum() / (2 * _volume(box))
    root = math.sqrt(math.pi)
    return torch.stack([recip, -alpha / root * (q * q).sum(),
                        -2 * alpha ** 3 / (3 * root) * (mu * mu).sum()])


def _exact_pme(pos, q, mu, box, mesh, p, alpha, tangents=()):
    """Energy parts, gradient and the Hessian applied to each tangent (pos, q, mu), in
    chunks of atoms: E = rho^T K rho / 2V, so with phi = K rho the gradient is that of
    <rho, phi> / V at fixed phi, and H v adds <rho, K rho_dot>."""
    n, m = len(q), math.prod(mesh)
    step = max(1, 3_000_000 // p ** 3)
    spans = [slice(i, i + step) for i in range(0, n, step)]
    inp = (pos, q, mu)
    values = lambda x: _footprint(*x, box, mesh, p)[1]  # noqa: E731
    rho = torch.zeros(m, dtype=torch.float64, device=pos.device)
    dots = [torch.zeros_like(rho) for _ in tangents]
    for c in spans:
        x = tuple(t[c] for t in inp)
        at, val = _footprint(*x, box, mesh, p)
        rho.index_add_(0, at.reshape(-1), val.reshape(-1))
        for dot, v in zip(dots, tangents):
            dval = torch.func.jvp(lambda a, b, d: values((a, b, d)), x, tuple(t[c] for t in v))[1]
            dot.index_add_(0, at.reshape(-1), dval.reshape(-1))
    phi = _convolve(rho, box, mesh, p, alpha)
    vol, root = _volume(box), math.sqrt(math.pi)
    energy = torch.stack([(rho * phi).sum() / (2 * vol), -alpha / root * (q * q).sum(),
                          -2 * alpha ** 3 / (3 * root) * (mu * mu).sum()])
    psis = [_convolve(dot, box, mesh, p, alpha) for dot in dots]
    cq, cm = 2 * alpha / root, 4 * alpha ** 3 / (3 * root)
    grad, hvp = [], [[] for _ in tangents]
    for c in spans:
        x = [t[c].clone().requires_grad_() for t in inp]
        at, val = _footprint(*x, box, mesh, p)
        g = torch.autograd.grad((val * phi[at]).sum(), x, create_graph=bool(tangents))
        grad.append([g[0].detach() / vol, g[1].detach() / vol - cq * q[c], g[2].detach() / vol - cm * mu[c]])
        for k, (v, psi) in enumerate(zip(tangents, psis)):
            t = sum((a * b[c]).sum() for a, b in zip(g, v)) + (val * psi[at]).sum()
            h = torch.autograd.grad(t, x, retain_graph=True)
            hvp[k].append([h[0] / vol, h[1] / vol - cq * v[1][c], h[2] / vol - cm * v[2][c]])
    join = lambda rows: [torch.cat(col) for col in zip(*rows)]  # noqa: E731
    return energy, join(grad), [join(h) for h in hvp]


def _pairs(pos, box, rc):
    """Ordered pairs within rc under the minimum image and their constant shifts."""
    ia, ja, shift = [], [], []
    side = torch.diagonal(box)
    for i in range(0, len(pos), 1024):
        d = pos[i:i + 1024, None] - pos[None]
        s = side * torch.round(d / side)
        r2 = ((d - s) ** 2).sum(-1)
        a, b = torch.nonzero((r2 < rc * rc) & (r2 > 0), as_tuple=True)
        ia.append(a + i)
        ja.append(b)
        shift.append(s[a, b])
    return torch.cat(ia), torch.cat(ja), torch.cat(shift)


def _thole_real(pos, q, mu, pol, pairs, alpha):
    """The Thole-damped real-space energy (damping constant 0.39)."""
    ia, ja, shift = pairs
    R = pos[ia] - pos[ja] - shift
    r = R.norm(dim=-1)
    gauss = torch.exp(-(alpha * r) ** 2) / (alpha * math.sqrt(math.pi))
    b0 = torch.special.erfc(alpha * r) / r
    b1 = (b0 + 2 * alpha ** 2 * gauss) / r ** 2
    b2 = (3 * b1 + (2 * alpha ** 2) ** 2 * gauss) / r ** 2
    u = 0.39 * r ** 3 / torch.sqrt(pol[ia] * pol[ja])
    b1 = b1 - torch.exp(-u) / r ** 3
    b2 = b2 - 3 * (1 + u) * torch.exp(-u) / r ** 5
    mi, mj = mu[ia], mu[ja]
    mir, mjr = (mi * R).sum(-1), (mj * R).sum(-1)
    return 0.5 * (q[ia] * q[ja] * b0 + (q[ia] * mjr - q[ja] * mir) * b1
                  + (mi * mj).sum(-1) * b1 - mir * mjr * b2).sum()


def _model_energy(pos, q, mu, pol, box, pairs, mesh, p, alpha):
    return (_parts_recip(pos, q, mu, box, mesh, p, alpha).sum()
            + _thole_real(pos, q, mu, pol, pairs, alpha) + ((mu * mu).sum(-1) / (2 * pol)).sum())


def _induced(pos, q, pol, box, pairs, mesh, p, alpha):
    """Self-consistent dipoles by conjugate gradients to 1e-11 of the right-hand side."""
    def slope(charges, m):
        m = m.clone().requires_grad_()
        return torch.autograd.grad(_model_energy(pos, charges, m, pol, box, pairs, mesh, p, alpha), m)[0]

    x = torch.zeros(len(q), 3, dtype=torch.float64, device=pos.device)
    r = -slope(q, x)
    z = pol[:, None] * r
    d, rz, stop = z, (r * z).sum(), 1e-11 * r.norm()
    for _ in range(200):
        if r.norm() < stop:
            break
        ad = slope(torch.zeros_like(q), d)
        a = rz / (d * ad).sum()
        x, r = x + a * d, r - a * ad
        z = pol[:, None] * r
        rz, old = (r * z).sum(), rz
        d = z + rz / old * d
    return x


def _features(pos, z, pairs):
    ia, ja, shift = pairs
    R = pos[ia] - pos[ja] - shift
    r = R.norm(dim=-1)
    t = r / R_FEAT
    env = 1 - 21 * t ** 5 + 35 * t ** 6 - 15 * t ** 7
    k = torch.arange(1, 9, dtype=torch.float64, device=pos.device)
    radial = math.sqrt(2 / R_FEAT) * torch.sin(math.pi * t[:, None] * k) * (env / r)[:, None]
    row = 2 * ia + (z[ja] <= 0).long()   # (atom, species of the neighbour)
    n = len(z)
    scal = torch.zeros(2 * n, 8, dtype=torch.float64, device=pos.device).index_add(0, row, radial)
    pull = (z[ja, None] * radial)[:, :, None] * (R / r[:, None])[:, None, :]
    vec = torch.zeros(2 * n, 8, 3, dtype=torch.float64, device=pos.device).index_add(0, row, pull)
    vec = vec.reshape(n, 16, 3)
    kind = torch.stack([z > 0, z <= 0], -1).double()
    return torch.cat([scal.reshape(n, 16), (vec * vec).sum(-1), kind], -1), vec


def _heads(theta, qtheta, z, feat, vec):
    """Charges and dipoles of the two perceptrons."""
    silu = torch.nn.functional.silu
    w1, b1, w2, b2, w3, b3 = torch.split(theta, [64 * 34, 64, 64 * 64, 64, 16 * 64, 16])
    h = silu(feat @ w1.reshape(64, 34).T + b1)
    w = silu(h @ w2.reshape(64, 64).T + b2) @ w3.reshape(16, 64).T + b3
    u1, c1, u2 = torch.split(qtheta, [64 * 34, 64, 64])
    c = silu(feat @ u1.reshape(64, 34).T + c1) @ u2
    return z + c - c.mean(), (w[:, :, None] * vec).sum(1)


def _exact_heads(case, s, mesh, p, alpha):
    pos, z, pol, box = (s[k].double() for k in ("pos", "q", "pol", "box"))
    theta, qtheta = (torch.tensor(s[k], dtype=torch.float32, device="cuda").double().requires_grad_()
                     for k in ("theta", "qtheta"))
    far, near = _pairs(pos, box, R_PAIR), _pairs(pos, box, R_FEAT)
    train = case["kind"] == "train"
    pos = pos.requires_grad_()
    feat, vec = _features(pos, z, near)
    q, mu = _heads(theta, qtheta, z, feat, vec)
    energy = _model_energy(pos, q, mu, pol, box, far, mesh, p, alpha)
    (slope,) = torch.autograd.grad(energy, pos, create_graph=train)
    if not train:
        return {"feat": feat.detach(), "vec": vec.detach(), "energy": energy.detach().reshape(1),
                "dU_dpos": slope, "q": q.detach(), "mu": mu.detach()}
    loss = (((energy - s["e_ref"]) / len(z)) ** 2).sum() + (slope - s["f_ref"].double()).square().mean()
    grad = torch.cat(torch.autograd.grad(loss, [theta, qtheta]))
    # Adam's first step: both moment estimates are the gradient's own
    new = torch.cat([theta, qtheta]).detach() - 3e-3 / 150 * grad / (grad.abs() + 1e-8)
    return {"loss": loss.detach().reshape(1), "grad": grad, "params": new}


def exact(case, seed):
    s = _inputs(case, seed)
    kind, p, alpha = case["kind"], case["order"], case["alpha"]
    box = s["box"]
    if kind == "batch":
        out, first = [], 0
        for b, n in enumerate(_batch_counts(case)):
            x = {k: s[k][first:first + n].double() for k in ("pos", "q", "mu", "v_pos", "v_q", "v_mu", "vf_pos")}
            first += n
            none = (x["vf_pos"], torch.zeros_like(x["q"]), torch.zeros_like(x["mu"]))
            e, g, h = _exact_pme(x["pos"], x["q"], x["mu"], box[b], _batch_mesh(n), p, alpha,
                                 [(x["v_pos"], x["v_q"], x["v_mu"]), none])
            out.append([e] + g + h[0] + h[1])
        cols = [torch.stack(c) if k == 0 else torch.cat(c) for k, c in enumerate(zip(*out))]
        names = ["energy"] + [stem.replace("X", x) for stem in ("dE_dX", "g_X", "gf_X") for x in ("pos", "q", "mu")]
        return dict(zip(names, cols))
    mesh = (case["mx"], case["my"], case["mz"])
    if kind in ("student", "train"):
        return _exact_heads(case, s, mesh, p, alpha)
    pos, q, mu = (s[k].double() for k in ("pos", "q", "mu"))
    if kind == "teacher":
        pol, pairs = s["pol"].double(), _pairs(pos, box, R_PAIR)
        m = _induced(pos, q, pol, box, pairs, mesh, p, alpha)
        pos = pos.requires_grad_()
        energy = _model_energy(pos, q, m, pol, box, pairs, mesh, p, alpha)
        return {"mu": m, "dU_dpos": torch.autograd.grad(energy, pos)[0]}
    tangents = [tuple(s[k].double() for k in ("v_pos", "v_q", "v_mu"))] if "v_pos" in s else []
    if kind == "force_loss":
        energy, grad, _ = _exact_pme(pos, q, mu, box, mesh, p, alpha)
        miss, n = (energy.sum() - s["e_ref"]) / len(q), len(q)
        v = 2 / (3 * n) * (grad[0] + s["f_ref"].double())
        loss = (miss ** 2).sum() + (grad[0] + s["f_ref"].double()).square().mean()
        h = _exact_pme(pos, q, mu, box, mesh, p, alpha,
                       [(v, torch.zeros_like(q), torch.zeros_like(mu))])[2][0]
        return [loss, grad[0], *[2 * miss / n * g + t for g, t in zip(grad, h)]]
    energy, grad, hvp = _exact_pme(pos, q, mu, box, mesh, p, alpha, tangents)
    if kind == "energy":
        return [energy.sum(), *grad]
    out = dict(zip(("energy", "dE_dpos", "dE_dq", "dE_dmu"), [energy] + grad))
    if tangents:
        out.update(zip(("g_pos", "g_q", "g_mu"), hvp[0]))
    if kind == "stress":
        cell = box.clone().requires_grad_()
        if math.prod(mesh) > 6_000_000:
            out["dE_dbox"] = None
        else:
            parts = _parts_recip(pos, q, mu, cell, mesh, p, alpha)
            out["dE_dbox"] = torch.autograd.grad(parts.sum(), cell)[0]
    return out
