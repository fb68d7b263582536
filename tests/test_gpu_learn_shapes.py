"""The learned start's kernels at the sizes where their tilings can go wrong,
against the oracle.

Features are defined bit by bit (a total order of neighbours, a sum in atom
order), so the test is exact equality: tile edges of the search (64 and 256
candidates, 16 atoms per workgroup), systems that share a workgroup, ties
(lattice points), coincident atoms, coordinates far from the origin, and atoms
at their system's centroid, whose offsets have no sure rounding until the
ordered sum is formed.
"""
import numpy as np
import pytest
import torch

from oracle import learn as OL
from paper_1810_03358_amd import learn as L
from tests.systems import make_system

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _points(n, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "lattice":                       # many equal distances, symmetric about the origin
        k = int(np.ceil(n ** (1 / 3)))
        g = np.stack(np.meshgrid(*[np.arange(k) - (k - 1) / 2] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
        return 1.5 * g[rng.permutation(len(g))[:n]]
    x = rng.normal(scale=8.0, size=(n, 3))
    if kind == "coincident":
        x[n // 2:] = x[: n - n // 2]
    if kind == "offset":                        # coordinates whose FP32 spacing exceeds a neighbour distance
        x += np.array([3.0e7, -2.0e7, 1.0e7])
    if kind == "line":                          # one direction, increasing gaps: far neighbours for the last atoms
        x = np.stack([np.cumsum(np.arange(n) * 0.1), np.zeros(n), np.zeros(n)], axis=1)
    return x


@pytest.mark.parametrize("kind", ["normal", "lattice", "coincident", "offset", "line"])
@pytest.mark.parametrize("sizes", [(1,), (2, 1, 3), (16, 17), (63, 64, 65), (255,), (256,), (257,), (272, 5, 9, 520),
                                   (769,)])
def test_features_at_the_edges_of_the_search(sizes, kind):
    systems = []
    for i, n in enumerate(sizes):
        rng = np.random.default_rng([n, i])
        systems.append(make_system(_points(n, kind, n + i), q=rng.uniform(-0.5, 0.5, n), sigma=rng.uniform(3, 4, n),
                                   eps=rng.uniform(0.05, 0.2, n)))
    sa = L.SystemArrays(systems, DEV)
    x = np.concatenate([s["x"] for s in systems])
    f, nb = L.features(sa, torch.tensor(x, dtype=torch.float64, device=DEV).contiguous(), want_neighbors=True)
    cat = lambda k: np.concatenate([s[k] for s in systems])  # noqa: E731
    fo, nbo = OL.features(x, cat("q"), cat("sigma"), cat("eps"), sa.sys_first_host)
    np.testing.assert_array_equal(nb.cpu().numpy(), nbo)
    np.testing.assert_array_equal(f.cpu().numpy().view(np.uint16), fo)


# rows of a wavefront (16) and of a workgroup (64) with remainders, and more
# row blocks than workgroups of the backward (256) and forward (512) kernels
@pytest.mark.parametrize("rows", [2, 14, 18, 62, 66, 130])
@pytest.mark.parametrize("shift", [0, 1])
def test_network_is_exact_on_exact_inputs_at_row_remainders(rows, shift):
    """shift = 1: features at an odd 2-byte offset, which the fused kernels'
    8-byte loads cannot read (the products run one by one)."""
    from tests.learn_exact import exact_case
    theta, fbits, T = exact_case(rows, 10 + rows)
    buf = torch.zeros(fbits.size + shift, dtype=torch.int16, device=DEV)
    xb = buf[shift:].view(rows, 128)
    xb.copy_(torch.tensor(fbits.view(np.int16)))
    net = L.Net(theta, device=DEV)
    X = OL.bf16_value(fbits)
    yo, _ = OL.forward(theta.astype(np.float64), X, emulate=True)
    np.testing.assert_array_equal(net.forward(xb).cpu().numpy().astype(np.float64), yo)
    loss = net.loss_grad(xb, torch.tensor(T, device=DEV))
    lo, go = OL.loss_grad(theta.astype(np.float64), X, T.astype(np.float64), emulate=True)
    assert float(loss.cpu()[0]) == pytest.approx(lo, rel=1e-6)
    np.testing.assert_array_equal(net.grad.cpu().numpy().astype(np.float64), go)


def test_network_over_several_row_blocks_per_workgroup():
    """Copies of one exact case: 520 row blocks for the forward pass, and 512 for
    the backward pass, where dY is the small case's times a power of two, so
    that every product and sum stays exact."""
    from tests.learn_exact import exact_case
    theta, fbits, T = exact_case(64, 5)
    rows = lambda a, k: np.tile(a, (k, 1))  # noqa: E731
    net = L.Net(theta, device=DEV)
    y = net.forward(torch.tensor(rows(fbits.view(np.int16), 520), device=DEV)).cpu().numpy().reshape(520, 64, 16)
    yo, _ = OL.forward(theta.astype(np.float64), OL.bf16_value(fbits), emulate=True)
    np.testing.assert_array_equal(y.astype(np.float64), np.broadcast_to(yo, y.shape))
    loss = net.loss_grad(torch.tensor(rows(fbits.view(np.int16), 512), device=DEV),
                         torch.tensor(rows(T, 512), device=DEV))
    lo, go = OL.loss_grad(theta.astype(np.float64), OL.bf16_value(rows(fbits, 512)), rows(T, 512).astype(np.float64),
                          emulate=True)
    assert float(loss.cpu()[0]) == pytest.approx(lo, rel=1e-6)
    np.testing.assert_array_equal(net.grad.cpu().numpy(), go.astype(np.float32))
