"""The work a program has this library do, as cases that can be timed.

Each case is one call (or one short sequence of calls) of the public Python
entry points on inputs made from a seed:

* ``eval``      energy and gradient of one system or of a batch on a context
                (a caller's own optimizer or sampler; also what every
                iteration of the built-in minimizers consists of)
* ``noalloc``   the same for one system without a context
* ``minimize``  a bounded number of iterations of a minimizer
* ``predict``   features, network and displaced start of the learned warm start
* ``train``     one minibatch step of its training loop

Inputs are chains with the parameters of the repository's workloads (bond
1.5 A, angle 109.5 degrees, q in [-0.5, 0.5], sigma in [3, 4] A, eps in
[0.05, 0.2] kcal/mol) in one of two shapes: ``coil``, a freely rotating chain
with 0.3 A of noise, the clash-laden start of a minimization; and ``fold``, a
dense chain (0.03 atoms/A^3) near its rest geometry with 0.05 A of noise, the
kind of point where a minimization spends most of its iterations.
"""
import math
import os

import numpy as np
import torch

import paper_1810_03358_amd as ff
from paper_1810_03358_amd import learn

COULOMB = 1389.38757 / 4.184
BOND, ANGLE = 1.5, math.radians(109.5)
ROW, ROWS, SPACING = 20, 5, 5.2          # fold: 20-atom rows, 5 x 5 rows a brick, 5.2 A apart
DEVICE = "cuda"


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one small chain at its start: latency and launches
        dict(name="eval_512_fp64", kind="eval", n=512, shape="coil", precision="fp64", torsions=False, links=0),
        # a caller that may not allocate: the system is packed on every call
        dict(name="noalloc_2311_fp32", kind="noalloc", n=2311, shape="coil", precision="fp32", torsions=True, links=0),
        # a protein-sized chain near a minimum, all term kinds, cross-links
        dict(name="eval_9973_fp64", kind="eval", n=9973, shape="fold", precision="fp64", torsions=True, links=6),
        # the same size in the mixed precision of the first part of a minimization
        dict(name="eval_10000_fp32", kind="eval", n=10000, shape="fold", precision="fp32", torsions=False, links=0),
        # the benchmark's size in both precisions: throughput of the pair sum
        dict(name="eval_50000_fp32", kind="eval", n=50000, shape="fold", precision="fp32", torsions=False, links=0),
        dict(name="eval_50000_fp64", kind="eval", n=50000, shape="fold", precision="fp64", torsions=False, links=0),
        # many uneven chains evaluated together
        dict(name="eval_batch96_fp64", kind="eval", n=4000, count=96, shape="fold", precision="fp64", torsions=False,
             links=0),
        # a small chain minimized from its clashing start
        dict(name="lbfgs_512_fp64", kind="minimize", n=512, shape="coil", precision="fp64", torsions=False, links=0,
             method="lbfgs", m=10, iters=30),
        # a protein-sized chain in mixed precision: the iterations after the clashes
        dict(name="lbfgs_10007_fp32", kind="minimize", n=10007, shape="fold", precision="fp32", torsions=False,
             links=0, method="lbfgs", m=10, iters=20),
        # many uneven chains minimized together in the precision of the end game
        dict(name="lbfgs_batch64_fp64", kind="minimize", n=4000, count=64, shape="fold", precision="fp64",
             torsions=False, links=0, method="lbfgs", m=10, iters=20),
        # the learned start of one protein-sized chain
        dict(name="predict_10000", kind="predict", n=10000, shape="coil"),
        # one training step of its network at the size the shipped weights were trained with
        dict(name="train_8192", kind="train", rows=8192),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choices(("eval", "batch", "noalloc", "minimize", "predict", "train"), (6, 2, 1, 3, 2, 2))[0]
    shape = rng.choice(("coil", "fold"))
    if kind == "train":
        return dict(kind="train", rows=size(256, 32768))
    if kind == "predict":
        case = dict(kind="predict", n=size(100, 10000), shape=shape)
        if rng.random() < 0.4:
            case.update(n=min(case["n"], 4000), count=rng.randint(2, 24))
        return case
    case = dict(kind=kind, n=size(150, 50000), shape=shape, precision=rng.choice(("fp64", "fp32")),
                torsions=rng.random() < 0.5, links=rng.choice((0, 0, 0, 4)))
    if kind == "batch":
        case.update(kind="eval", n=size(400, 4000), count=rng.randint(3, 96))
    elif kind == "noalloc":
        case.update(n=size(150, 20000))
    elif kind == "minimize":
        case.update(n=size(150, 10000), method=rng.choice(("lbfgs", "lbfgs", "cg", "gd")), m=rng.choice((3, 10)),
                    iters=rng.randint(6, 16), links=0)
        if rng.random() < 0.4:
            case.update(n=size(400, 4000), count=rng.randint(3, 48))
    return case


# ------------------------------------------------------------------- inputs
def _coil(n, rng):
    """Rest geometry of a freely rotating chain (prefix products of the bond
    rotations)."""
    phi = rng.uniform(-math.pi, math.pi, size=n)
    c, s, ct, st = np.cos(phi), np.sin(phi), -math.cos(ANGLE), math.sin(ANGLE)
    rot = np.empty((n, 3, 3))
    rot[:, 0, 0], rot[:, 0, 1], rot[:, 0, 2] = ct, -st, 0.0
    rot[:, 1, 0], rot[:, 1, 1], rot[:, 1, 2] = c * st, c * ct, -s
    rot[:, 2, 0], rot[:, 2, 1], rot[:, 2, 2] = s * st, s * ct, c
    step = 1
    while step < n:
        rot[step:] = rot[:-step] @ rot[step:]
        step *= 2
    x = np.zeros((n, 3))
    x[1:] = np.cumsum(BOND * rot[:n - 1, :, 0], axis=0)
    return x


def _fold(n):
    """Rest geometry of a dense chain: zigzag rows laid to and fro, brick
    after brick of rows laid to and fro."""
    row, k = np.divmod(np.arange(n), ROW)
    brick, r = np.divmod(row, ROWS * ROWS)
    rz, ry = np.divmod(r, ROWS)
    ry = np.where(rz % 2 == 0, ry, ROWS - 1 - ry)
    side = max(1, round((brick[-1] + 1) ** (1.0 / 3.0)))
    bz, rest = np.divmod(brick, side * side)
    by, bx = np.divmod(rest, side)
    by = np.where(bz % 2 == 0, by, side - 1 - by)
    bx = np.where((by + bz) % 2 == 0, bx, side - 1 - bx)
    rz = np.where(brick % 2 == 0, rz, ROWS - 1 - rz)
    pos = np.where(row % 2 == 0, k, ROW - 1 - k)
    adv, amp = BOND * math.sin(ANGLE / 2), BOND * math.cos(ANGLE / 2)
    return np.stack([bx * (ROW * adv + 4.0) + pos * adv,
                     (by * ROWS + ry) * SPACING + (k % 2) * amp,
                     (bz * ROWS + rz) * SPACING], axis=1)


def _angle(x, t):
    u, v = x[t[:, 0]] - x[t[:, 1]], x[t[:, 2]] - x[t[:, 1]]
    return np.arctan2(np.linalg.norm(np.cross(u, v), axis=1), (u * v).sum(axis=1))


def _system(case, n, rng):
    """A system dict and its coordinates."""
    rest = _coil(n, rng) if case["shape"] == "coil" else _fold(n)
    k = np.arange(n)
    bonds = np.stack([k[:-1], k[1:]], axis=1)
    angles = np.stack([k[:-2], k[1:-1], k[2:]], axis=1)
    for _ in range(case.get("links", 0)):
        i = int(rng.integers(1, n // 4))
        j = int(rng.integers(n // 2 + 1, n - 1))
        bonds = np.concatenate([bonds, [[i, j]]])
        angles = np.concatenate([angles, [[i - 1, i, j], [i, j, j + 1]]])
    nd = n - 3 if case.get("torsions") else 0
    q = rng.uniform(-0.5, 0.5, size=n)
    system = dict(
        n_atoms=n, q=q - q.mean(), sigma=rng.uniform(3.0, 4.0, size=n), eps=rng.uniform(0.05, 0.2, size=n),
        bonds=bonds.astype(np.int32), bond_k=np.full(len(bonds), 300.0),
        bond_r0=np.linalg.norm(rest[bonds[:, 0]] - rest[bonds[:, 1]], axis=1),
        angles=angles.astype(np.int32), angle_k=np.full(len(angles), 50.0), angle_t0=_angle(rest, angles),
        dihedrals=(np.arange(nd)[:, None] + np.arange(4)).astype(np.int32),
        dihedral_v=rng.uniform(-2.0, 2.0, size=(nd, 4)), coulomb_c=COULOMB)
    x = rest + rng.normal(scale=0.3 if case["shape"] == "coil" else 0.05, size=(n, 3))
    return system, x - x.mean(axis=0)


def _sizes(case):
    """Atoms of each system: batches are log-uniform from 200 to n."""
    count = case.get("count", 0)
    if not count:
        return [case["n"]]
    rng = np.random.default_rng([count, case["n"]])
    return [int(round(v)) for v in np.exp(rng.uniform(math.log(200), math.log(case["n"]), size=count))]


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    pairs = [_system(case, n, rng) for n in _sizes(case)]
    x = torch.tensor(np.concatenate([x for _, x in pairs]), dtype=torch.float64, device=DEVICE)
    systems = [s for s, _ in pairs]
    return (systems if case.get("count") else systems[0]), x


def _train_inputs(case, seed):
    """Dataset rows (features: unit-scale values, zero padding), targets, the
    minibatch's row numbers, and Adam's moments as after some steps."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    rows = case["rows"]
    feats = torch.randn((2 * rows, learn.FEATURES), generator=g, device=DEVICE) * 0.5
    feats[:, 120:] = 0.0
    target = torch.randn((2 * rows, 3), generator=g, device=DEVICE) * 3.0
    idx = torch.randperm(2 * rows, generator=g, device=DEVICE)[:rows].to(torch.int32)
    m = torch.randn(learn.param_count(), generator=g, device=DEVICE) * 1e-2
    v = (torch.rand(learn.param_count(), generator=g, device=DEVICE) + 0.5) * 1e-3
    return feats.to(torch.bfloat16), target, idx, m, v


def _weights():
    path = os.path.join(os.path.dirname(os.path.abspath(ff.__file__)), "weights", "warmstart.npz")
    with np.load(path, allow_pickle=False) as z:
        return z["theta"].astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        feats, target, idx, m, v = _train_inputs(case, seed)
        net = learn.Net(_weights(), device=DEVICE)
        net.m.copy_(m)
        net.v.copy_(v)
        net.step = 100
        rows = case["rows"]
        return dict(case=case, net=net, X=feats.view(torch.int16), T=target, idx=idx,
                    fx=torch.empty((rows, learn.FEATURES), dtype=torch.int16, device=DEVICE),
                    tx=torch.empty((rows, 3), dtype=torch.float32, device=DEVICE),
                    loss=torch.empty(1, dtype=torch.float32, device=DEVICE))
    system, x = _inputs(case, seed)
    if kind == "predict":
        sa = learn.SystemArrays(system if case.get("count") else [system], DEVICE)
        return dict(case=case, sa=sa, net=learn.Net(_weights(), device=DEVICE), x=x)
    if kind == "noalloc":
        return dict(case=case, system=system, x=x, e=torch.empty(1, dtype=torch.float64, device=DEVICE),
                    g=torch.empty_like(x))
    return dict(case=case, ctx=ff.Context(system, m_max=case.get("m", 0), device=DEVICE), x=x)


# --------------------------------------------------------------------- a pass
def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "eval":
        return state["ctx"].energy_grad(state["x"], case["precision"])
    if kind == "noalloc":
        return ff.energy_grad_noalloc(state["system"], state["x"], state["e"], state["g"], case["precision"])
    if kind == "minimize":
        x = state["x"].clone()
        res = state["ctx"].minimize(x, case["method"], m=case["m"], max_iter=case["iters"],
                                    precision=case["precision"])
        res = res if isinstance(res, list) else [res]
        out = {k: np.array([r[k] for r in res]) for k in ("energy", "grad_inf", "grad_2", "iters", "evals", "term")}
        out["x"] = x
        return out
    if kind == "predict":
        feats = learn.features(state["sa"], state["x"])
        y = state["net"].forward(feats)
        return dict(features=feats, displacement=y, start=learn.displace(state["x"], y, 0.5))
    net = state["net"]
    learn.gather_rows(state["X"], state["idx"], state["fx"])
    learn.gather_rows(state["T"], state["idx"], state["tx"])
    net.loss_grad(state["fx"], state["tx"], state["loss"])
    net.adam_step(1e-3)
    return dict(loss=state["loss"], grad=net.grad, theta=net.theta, m=net.m, v=net.v)


def work(case):
    kind = case["kind"]
    params = 128 * 128 * 2 + 128 * 16
    if kind == "train":
        rows = case["rows"]
        # rows read once (features, targets, indices), parameters and moments read and written
        return dict(bytes=rows * (256 + 12 + 4) + 35088 * (4 + 2 + 3 * 8 + 4),
                    flops=rows * (2 * params + 2 * (params + 128 * 128 + 128 * 16)))
    sizes = _sizes(case)
    n, pairs = sum(sizes), sum(k * (k - 1) // 2 for k in sizes)
    if kind == "predict":
        return dict(bytes=n * (24 + 24 + 256 + 64 + 24) + params * 2, flops=2 * pairs * 8 + n * 2 * params)
    # coordinates, gradient, parameters and topology once an evaluation
    one = dict(bytes=n * (24 + 24 + 24 + 24 + 28), flops=38 * pairs)
    if kind != "minimize":
        return one
    # two evaluations an iteration and, for L-BFGS, the stored pairs read for
    # the direction and for the products of the new pair
    vectors = 6 + (4 * case["m"] if case["method"] == "lbfgs" else 2)
    return dict(bytes=case["iters"] * (2 * one["bytes"] + 24 * n * vectors), flops=case["iters"] * 2 * one["flops"])


# ------------------------------------------------------------- in 64 bits
def _exact_energy(s, x):
    """Energy and gradient of one system as plain double-precision torch."""
    n = s["n_atoms"]
    dev = x.device
    t = lambda k: torch.tensor(s[k], dtype=torch.float64, device=dev)  # noqa: E731
    q, sig3, eps = t("q"), t("sigma") ** 1.5, t("eps").sqrt()
    ex = torch.tensor(np.concatenate([s["bonds"], s["angles"][:, [0, 2]]]), dtype=torch.long, device=dev)
    ex = torch.cat([ex, ex.flip(1)])
    ex = ex[ex[:, 0].argsort()]
    first = ex[:, 0].contiguous()
    energy = torch.zeros((), dtype=torch.float64, device=dev)
    grad = torch.empty_like(x)
    rows = max(1, min(n, 30_000_000 // n))
    for a in range(0, n, rows):
        b = min(n, a + rows)
        d = [x[None, :, c] - x[a:b, None, c] for c in range(3)]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        r2[torch.arange(b - a, device=dev), torch.arange(a, b, device=dev)] = math.inf
        lo, hi = torch.searchsorted(first, torch.tensor([a, b], device=dev)).tolist()
        r2[ex[lo:hi, 0] - a, ex[lo:hi, 1]] = math.inf
        inv2 = 1.0 / r2
        s6 = (sig3[a:b, None] * sig3[None, :]) ** 2 * inv2 ** 3
        e4 = 4.0 * eps[a:b, None] * eps[None, :] * s6
        ec = s["coulomb_c"] * q[a:b, None] * q[None, :] * inv2.sqrt()
        energy += 0.5 * (e4 * (s6 - 1.0) + ec).sum()
        f = (e4 * (12.0 * s6 - 6.0) + ec) * inv2
        for c in range(3):
            grad[a:b, c] = (f * d[c]).sum(dim=1)
    xb = x.clone().requires_grad_(True)
    i = torch.tensor(s["bonds"], dtype=torch.long, device=dev)
    r = (xb[i[:, 0]] - xb[i[:, 1]]).norm(dim=1)
    bonded = (t("bond_k") * (r - t("bond_r0")) ** 2).sum()
    i = torch.tensor(s["angles"], dtype=torch.long, device=dev)
    u, v = xb[i[:, 0]] - xb[i[:, 1]], xb[i[:, 2]] - xb[i[:, 1]]
    th = torch.atan2(torch.linalg.cross(u, v).norm(dim=1), (u * v).sum(dim=1))
    bonded = bonded + (t("angle_k") * (th - t("angle_t0")) ** 2).sum()
    if len(s["dihedrals"]):
        i = torch.tensor(s["dihedrals"], dtype=torch.long, device=dev)
        f, g, h = xb[i[:, 0]] - xb[i[:, 1]], xb[i[:, 1]] - xb[i[:, 2]], xb[i[:, 3]] - xb[i[:, 2]]
        na, nb = torch.linalg.cross(f, g), torch.linalg.cross(h, g)
        phi = torch.atan2((torch.linalg.cross(nb, na) * g).sum(dim=1) / g.norm(dim=1), (na * nb).sum(dim=1))
        w = t("dihedral_v")
        bonded = bonded + 0.5 * (w[:, 0] * (1 + torch.cos(phi)) + w[:, 1] * (1 - torch.cos(2 * phi))
                                 + w[:, 2] * (1 + torch.cos(3 * phi)) + w[:, 3] * (1 - torch.cos(4 * phi))).sum()
    bonded.backward()
    return (energy + bonded.detach()).reshape(1), grad + xb.grad


def _exact_features(s, x):
    """Feature rows of one system before rounding."""
    n = s["n_atoms"]
    dev = x.device
    own = torch.stack([torch.tensor(s["q"], device=dev), torch.tensor(s["sigma"], device=dev) - 3.5,
                       10.0 * torch.tensor(s["eps"], device=dev)], dim=1)
    k = min(learn.NEIGHBORS, n - 1)
    out = torch.zeros((n, learn.FEATURES), dtype=torch.float64, device=dev)
    out[:, :3] = own
    rows = max(1, 20_000_000 // n)
    for a in range(0, n, rows):
        b = min(n, a + rows)
        d2 = sum((x[None, :, c] - x[a:b, None, c]) ** 2 for c in range(3))
        d2[torch.arange(b - a, device=dev), torch.arange(a, b, device=dev)] = math.inf
        val, j = torch.topk(d2, k, dim=1, largest=False, sorted=True)
        near = torch.cat([(x[j] - x[a:b, None]) / 4.0, (val.sqrt() / 4.0)[:, :, None], own[j]], dim=2)
        out[a:b, 3:3 + 7 * k] = near.reshape(b - a, 7 * k)
    c = x - x.mean(dim=0)
    at = 3 + 7 * learn.NEIGHBORS
    out[:, at:at + 3] = c / 16.0
    out[:, at + 3] = c.norm(dim=1) / 16.0
    out[:, at + 4] = n / 4096.0
    return out


def _exact_layers(dev):
    w = torch.tensor(_weights(), device=dev).double()
    parts = torch.split(w, [128 * 128, 128, 128 * 128, 128, 128 * 16, 16])
    return [(parts[2 * k].reshape(128, -1).clone(), parts[2 * k + 1].clone()) for k in range(3)]


def _exact_network(layers, rows):
    (w1, b1), (w2, b2), (w3, b3) = layers
    return torch.relu(torch.relu(rows @ w1 + b1) @ w2 + b2) @ w3 + b3


def exact(case, seed):
    kind = case["kind"]
    if kind == "minimize":
        return None
    if kind == "train":
        feats, target, idx, m, v = _train_inputs(case, seed)
        layers = [(w.requires_grad_(True), b.requires_grad_(True)) for w, b in _exact_layers(DEVICE)]
        y = _exact_network(layers, feats[idx.long()].double())
        loss = ((y[:, :3] - target[idx.long()].double()) ** 2).mean()
        loss.backward()
        g = torch.cat([p.grad.reshape(-1) for layer in layers for p in layer])
        m, v = 0.9 * m.double() + 0.1 * g, 0.999 * v.double() + 0.001 * g * g
        theta = torch.tensor(_weights(), device=DEVICE).double()
        theta = theta - 1e-3 * (m / (1 - 0.9 ** 101)) / ((v / (1 - 0.999 ** 101)).sqrt() + 1e-8)
        return dict(loss=loss.detach().reshape(1), grad=g, theta=theta, m=m, v=v)
    system, x = _inputs(case, seed)
    systems, at, parts = (system if case.get("count") else [system]), 0, []
    for s in systems:
        parts.append((s, x[at:at + s["n_atoms"]]))
        at += s["n_atoms"]
    if kind == "predict":
        y = _exact_network(_exact_layers(DEVICE), torch.cat([_exact_features(s, p) for s, p in parts]))
        return dict(features=None, displacement=y, start=x + 0.5 * y[:, :3])
    got = [_exact_energy(s, p) for s, p in parts]
    return torch.cat([e for e, _ in got]), torch.cat([g for _, g in got])
