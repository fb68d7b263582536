"""Features of the learned start for points and arrays that ordinary chains do
not have, exactly as the oracle defines them."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import learn as OL
from paper_1810_03358_amd import _native as N
from paper_1810_03358_amd import learn as L
from synth import chain_system
from tests.systems import make_system

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _system(x, seed):
    n, rng = len(x), np.random.default_rng(seed)
    return make_system(x, q=rng.uniform(-0.5, 0.5, n), sigma=rng.uniform(3, 4, n), eps=rng.uniform(0.05, 0.2, n))


def _oracle(s):
    return OL.features(s["x"], s["q"], s["sigma"], s["eps"], [0, s["n_atoms"]])


# squares of these distances are finite in FP64 and, above about 1.8e19, not in
# FP32, in which the search makes its first pass
@pytest.mark.parametrize("far", [1e15, 1e18, 1e19, 1e20, 1e25, 1e30])
@pytest.mark.parametrize("kind", ["first", "third", "every other", "halves"])
def test_far_apart_atoms_keep_their_neighbours(far, kind):
    """More atoms than one tile of the search (256); `far` away lie the first or
    third atom of some groups of four (which one wavefront searches), or a
    cluster of half of the atoms: every other one, or the second half and atom 1
    (whose neighbours then lie in tiles that hold none for atom 0)."""
    n, rng = 1030 if kind == "halves" else 600, np.random.default_rng(3)
    x = rng.normal(scale=8.0, size=(n, 3))
    if kind in ("every other", "halves"):
        at = np.arange(1, n, 2) if kind == "every other" else np.r_[1, 512:n]
        x[at] = far * np.array([1.0, -0.5, 0.25]) + rng.normal(scale=far * 1e-12 + 8.0, size=(len(at), 3))
    else:
        at = np.arange(0 if kind == "first" else 2, n, 40)
        x[at] = far * (1.0 + np.arange(len(at))[:, None]) * np.array([1.0, 0.5, -0.25])
    s = _system(x, 4)
    print(f"features far={far} {kind}", flush=True)
    f, nb = L.features(L.SystemArrays([s], DEV), torch.tensor(x, device=DEV), want_neighbors=True)
    fo, nbo = _oracle(s)
    np.testing.assert_array_equal(nb.cpu().numpy(), nbo)
    np.testing.assert_array_equal(f.cpu().numpy().view(np.uint16), fo)


@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 15, 17, 300])
def test_features_go_to_any_16_bit_address(n, shift):
    """The output array may begin at any multiple of two bytes; nothing before or
    behind it is written."""
    s = chain_system(n, 8)
    sa = L.SystemArrays([s], DEV)
    x = torch.tensor(s["x"], dtype=torch.float64, device=DEV).contiguous()
    buf = torch.full((n * L.FEATURES + 8,), 0x1234, dtype=torch.int16, device=DEV)
    print(f"features n={n} at {2 * shift} bytes", flush=True)
    p = lambda t, skip=0: C.c_void_p(t.data_ptr() + skip)  # noqa: E731
    assert N.load().ff_learn_features(1, n, p(x), p(sa.q), p(sa.sigma), p(sa.eps), p(sa.sys_first), p(sa.atom_sys),
                                      p(buf, 2 * shift), None, C.c_void_p(0)) == 0
    torch.cuda.synchronize()
    got = buf.cpu().numpy().view(np.uint16)
    end = shift + n * L.FEATURES
    np.testing.assert_array_equal(got[shift:end].reshape(n, L.FEATURES), _oracle(s)[0])
    assert (got[:shift] == 0x1234).all() and (got[end:] == 0x1234).all()


# from 640 systems of at most 16 atoms on average 16 share a centroid workgroup:
# by 16 lanes up to 16 atoms, a wavefront up to 64, the whole workgroup above
@pytest.mark.parametrize("sizes", [(1,) * 640, (3,) * 400 + (700,) + (1, 2) * 130, (16,) * 641, (16,) * 639,
                                   (15, 16, 17, 1) * 4 + (3,) * 320 + (64, 65) + (2,) * 333, (2, 64, 66, 20) * 2])
@pytest.mark.parametrize("kind", ["normal", "symmetric", "offset"])
def test_features_of_many_small_systems(sizes, kind):
    systems = []
    for k, n in enumerate(sizes):
        x = np.random.default_rng([n, k]).normal(scale=8.0, size=(n, 3))
        if kind == "symmetric":                 # centroid at an atom or between two, whose offsets nearly vanish
            x[n // 2:] = -x[: n - n // 2]
        systems.append(_system(x + (3.0e7 if kind == "offset" else 0.0), k))
    sa = L.SystemArrays(systems, DEV)
    x = np.concatenate([s["x"] for s in systems])
    print(f"features of {len(sizes)} systems, {kind}", flush=True)
    f, nb = L.features(sa, torch.tensor(x, device=DEV), want_neighbors=True)
    cat = lambda k: np.concatenate([s[k] for s in systems])  # noqa: E731
    fo, nbo = OL.features(x, cat("q"), cat("sigma"), cat("eps"), sa.sys_first_host)
    np.testing.assert_array_equal(nb.cpu().numpy(), nbo)
    np.testing.assert_array_equal(f.cpu().numpy().view(np.uint16), fo)
