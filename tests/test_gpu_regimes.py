"""FP64 evaluations on both sides of every line that the default tilings draw,
against the FP64 oracle.

FP64 chunks are a quarter, a half or the whole of a j-tile, so that they make
at least 512 wavefronts (fp64_parts below restates the rule), and several tiles
in larger systems; batches share workgroups and, past 4,096 of them, walk the
chunks in more than one round.

Gates: energies to 1e-11 relative, as everywhere; a gradient component to 2^-44
of the summed absolute pair forces on its atom (two evaluations of some 32
rounded operations a pair are 2^-47, the sums over a few hundred chunks the
rest) plus 1e-12 of the largest component for the bonded terms.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1810_03358_amd as ff
from oracle.energy import abs_pair_force
from tests.systems import crosslinked_chain, torsion_chain

pytestmark = pytest.mark.gpu
BLOCK, WAVES = 128, 1           # batches: tile configuration 9


def units(n, block):
    """Pairs of an I-block and a 64-atom tile."""
    nb = -(-n // block)
    return nb * (nb + 1) // 2 * (block // 64)


def fp64_parts(n_units, waves):
    """Parts that a one-tile FP64 chunk is cut into."""
    parts = 1
    while parts < 4 and n_units * waves * parts < 512:
        parts *= 2
    return parts


class Reference:
    def __init__(self):
        self.known = {}

    def __call__(self, make, n, seed):
        key = make.__name__, n, seed
        if key not in self.known:
            s = make(n, seed)
            self.known[key] = (s, *oracle.energy_grad(s, s["x"]), abs_pair_force(s, s["x"])[:, None])
        return self.known[key]


@pytest.fixture(scope="module")
def reference():
    return Reference()


def _check(refs, tiling=None):
    """One context over the reference systems; returns its tiling."""
    ctx = ff.Context([r[0] for r in refs] if len(refs) > 1 else refs[0][0], m_max=0, tiling=tiling)
    x = torch.tensor(np.concatenate([r[0]["x"].reshape(-1, 3) for r in refs]), dtype=torch.float64, device="cuda")
    e, g = ctx.energy_grad(x, "fp64")
    e, g, used = e.cpu().numpy(), g.cpu().numpy(), ctx.tiling
    ctx.close()
    at = 0
    for k, (s, e_ref, g_ref, pairs) in enumerate(refs):
        g_ref = np.asarray(g_ref).reshape(-1, 3)
        mine, at = g[at:at + s["n_atoms"]], at + s["n_atoms"]
        top = np.abs(g_ref).max()
        assert abs(e[k] - e_ref) <= 1e-11 * abs(e_ref), k
        bound = 2.0 ** -44 * pairs + 1e-12 * top
        assert np.all(np.abs(mine - g_ref) <= bound), (k, np.abs(mine - g_ref).max())
    return used


@pytest.mark.parametrize("n,parts", [(1280, 4), (1281, 2), (1792, 2), (1793, 1)])
def test_single_systems_across_the_split(reference, n, parts):
    """256-atom blocks of four wavefronts."""
    assert fp64_parts(units(n, 256), 4) == parts
    print(f"n={n} parts={parts}", flush=True)
    assert _check([reference(torsion_chain, n, 5)]) == (1, 1, 1)


# chains by size; the sizes repeat, so that the oracle evaluates each once
@pytest.mark.parametrize("sizes,parts,chunk64", [
    ((1000, 450, 64, 700), 4, 1), ((1000,) * 3 + (129,) * 2, 4, 1), ((1000,) * 3 + (450,) * 2, 2, 1),
    ((1000,) * 7, 2, 1), ((1000,) * 7 + (129,) * 2, 1, 1), ((1000, 450, 64, 700) * 9, 1, 1),
    ((1000,) * 240 + (450,), 1, 1), ((1000,) * 277 + (64,) * 20, 1, 1), ((1000,) * 277 + (64,) * 28, 1, 4),
    ((4100, 1000) * 18, 1, 4)], ids=lambda v: f"{len(v)}" if isinstance(v, tuple) else str(v))
def test_batches_across_the_rules(reference, sizes, parts, chunk64):
    total = sum(units(n, BLOCK) for n in sizes)
    assert (total >= 20000) == (chunk64 == 4) and (chunk64 == 4 or fp64_parts(total, WAVES) == parts)
    print(f"batch of {len(sizes)}, {total} tiles", flush=True)
    assert _check([reference(torsion_chain, n, 5) for n in sizes]) == (9, 4, chunk64)


def test_the_batches_hit_every_regime():
    """Quarters, halves, whole tiles, more chunks than 4,096 workgroups of four hold."""
    seen = {fp64_parts(sum(units(n, BLOCK) for n in s), WAVES)
            for s in ((1000, 450, 64, 700), (1000,) * 7, (1000,) * 7 + (129,) * 2)}
    assert seen == {4, 2, 1}
    assert 16384 < units(1000, BLOCK) * 240 < 20000


@pytest.mark.parametrize("cfg", list(range(len(ff.tile_configs()))))
def test_whole_one_tile_chunks_of_every_configuration(reference, cfg):
    t = ff.tile_configs()[cfg]
    assert fp64_parts(units(4100, t[0]), t[3]) == 1
    print(f"cfg={cfg}", flush=True)
    _check([reference(crosslinked_chain, 4100, 7)], (cfg, 1, 1))


@pytest.mark.parametrize("n,tiling", [
    (12287, (1, 1, 1)), (12288, (9, 1, 1)), (14500, (9, 1, 1)), (14501, (9, 1, 2)), (19999, (9, 1, 2)),
    (20000, (8, 1, 2)), (33000, (8, 2, 2)), (41000, (8, 2, 6)), (50001, (8, 2, 8))])
def test_default_tilings_of_large_systems(reference, n, tiling):
    print(f"n={n}", flush=True)
    assert _check([reference(crosslinked_chain, n, 9)]) == tiling
