"""The tiling that the library chooses by itself, from the workspace it asks for
(host side only): that of the named tiling, at the edges of each rule."""
import ctypes as C

import pytest

import paper_1810_03358_amd as ff
from paper_1810_03358_amd import _native as N
from synth import chain_system


@pytest.fixture(scope="module")
def chains():
    made = {}

    def get(n):
        if n not in made:
            made[n] = ff.HostSystem(chain_system(n, 1))
        return made[n]
    return get


def _bytes(hosts, tiling=None):
    lib, n = N.load(), len(hosts)
    arr = (N.FFSystem * n)(*[h.c for h in hosts])
    if tiling is None:
        return lib.ff_workspace_bytes_batch(arr, n, 0)
    return lib.ff_workspace_bytes_tiled(arr, n, 0, *tiling)


@pytest.mark.parametrize("n,tiling", [
    (1024, (0, 1, 1)), (1025, (1, 1, 1)), (12287, (1, 1, 1)), (12288, (9, 1, 1)), (14500, (9, 1, 1)),
    (14501, (9, 1, 2)), (19999, (9, 1, 2)), (20000, (8, 1, 2)), (32767, (8, 1, 2)), (32768, (8, 2, 2)),
    (40000, (8, 2, 2)), (40001, (8, 2, 6)), (49999, (8, 2, 6)), (50000, (8, 2, 8)), (60000, (8, 2, 8))])
def test_single_systems(chains, n, tiling):
    want = _bytes([chains(n)], tiling)
    assert want > 0 and _bytes([chains(n)]) == want


# 1,000 atoms are 72 tiles of 128-atom blocks, 4,000 atoms 1,056
@pytest.mark.parametrize("n,count,chunk64", [(1000, 2, 1), (1000, 277, 1), (1000, 278, 4), (4000, 18, 1), (4000, 19, 4),
                                             (4000, 100, 4), (50000, 2, 4)])
def test_batches(chains, n, count, chunk64):
    """Batches whose tiles fill the chip keep FP64 chunks of four tiles, and
    with them the workspace of four: one-tile chunks would ask for 16 % (4,000
    atoms each) to 68 % (50,000) more."""
    hosts = [chains(n)] * count
    assert _bytes(hosts) == _bytes(hosts, (9, 4, chunk64)) != _bytes(hosts, (9, 4, 5 - chunk64))
