"""FP64 evaluations of systems whose chunks are parts of a j-tile, against the
FP64 oracle.

Where one-tile chunks would be too few to fill the chip the FP64 kernel walks
half or quarter tiles, with a j-side partial row each; the sizes lie on both
sides of 64-atom tiles and of the rule's steps (a quarter of a tile up to about
1,000 atoms, a half up to about 2,800, whole tiles above; batches by their
total).  Splitting only reorders FP64 sums, so the gates are those of every
tiling: energy and gradient to 1e-11 relative (gradient: of its largest
component).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1810_03358_amd as ff
from tests.systems import crosslinked_chain, torsion_chain

pytestmark = pytest.mark.gpu


def _eval(systems, xs):
    ctx = ff.Context(systems, m_max=0)
    x = torch.tensor(np.concatenate([np.asarray(x).reshape(-1, 3) for x in xs]), dtype=torch.float64, device="cuda")
    e, g = ctx.energy_grad(x, "fp64")
    torch.cuda.synchronize()
    out = e.cpu().numpy(), g.cpu().numpy()
    ctx.close()
    return out


def _check(s, e, g):
    e_ref, g_ref = oracle.energy_grad(s, s["x"])
    assert abs(e - e_ref) <= 1e-11 * abs(e_ref)
    np.testing.assert_allclose(g.reshape(-1, 3), np.asarray(g_ref).reshape(-1, 3), rtol=0,
                               atol=1e-11 * np.abs(g_ref).max())


@pytest.mark.parametrize("n", [63, 64, 65, 129, 449, 512, 1023, 1024, 1025, 1281, 2049, 3001])
@pytest.mark.parametrize("chain", [torsion_chain, crosslinked_chain])
def test_sizes_across_the_split(n, chain):
    if chain is crosslinked_chain and n < 449:
        pytest.skip("no room for exclusions more than 64 atoms apart")
    s = chain(n, 7 + n)
    print(f"{chain.__name__} n={n}", flush=True)
    e, g = _eval([s], [s["x"]])
    _check(s, e[0], g)


@pytest.mark.parametrize("sizes", [(5, 63, 65), (130, 64, 200, 1), (700, 450, 512, 64, 1300)])
def test_batches_across_the_split(sizes):
    systems = [torsion_chain(n, 90 + k) for k, n in enumerate(sizes)]
    print("batch", sizes, flush=True)
    e, g = _eval(systems, [s["x"] for s in systems])
    at = 0
    for k, s in enumerate(systems):
        _check(s, e[k], g[at:at + sizes[k]])
        at += sizes[k]


@pytest.mark.parametrize("n", [512, 1500])
@pytest.mark.parametrize("pair", [(10, 40), (10, 300)], ids=["same tile", "tiles without exclusions"])
def test_coincident_atoms_do_not_spread(n, pair):
    """Two coincident atoms make the energy and their own gradients not finite
    and leave every other atom's gradient alone."""
    s = torsion_chain(n, 3)
    x = np.array(s["x"]).reshape(-1, 3)
    x[pair[1]] = x[pair[0]]
    s = dict(s, x=x)
    print(f"coincident {pair} n={n}", flush=True)
    e, g = _eval([s], [x])
    with np.errstate(all="ignore"):
        _, g_ref = oracle.energy_grad(s, x)
    g_ref = np.asarray(g_ref).reshape(-1, 3)
    other = np.setdiff1d(np.arange(n), pair)
    assert not np.isfinite(e[0]) and not np.isfinite(g[list(pair)]).any()
    assert np.isfinite(g_ref[other]).all()
    np.testing.assert_allclose(g[other], g_ref[other], rtol=0, atol=1e-11 * np.abs(g_ref[other]).max())
