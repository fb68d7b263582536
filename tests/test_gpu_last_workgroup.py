"""Reductions that a pass's last workgroup makes: repeated evaluations and
minimizations give the same bits, at one workgroup per system, at tile edges
and in batches whose systems finish in any order, and agree with the oracle.

The finalize and accept passes count their workgroups per system; a count that
is lost, kept from one pass to the next or read before the partials are in
memory shows as a result that differs between repeats.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1810_03358_amd as ff
from tests.systems import torsion_chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(3,), (64,), (65,), (300,), (2049,), (1, 700, 64, 65, 3, 1300)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_repeats_are_equal(sizes, prec):
    systems = [torsion_chain(n, 20 + k) for k, n in enumerate(sizes)]
    x = torch.tensor(np.concatenate([np.asarray(s["x"]).reshape(-1, 3) for s in systems]), dtype=torch.float64,
                     device="cuda")
    print(sizes, prec, flush=True)
    ctx = ff.Context(systems, m_max=4)
    e0, g0 = (t.cpu().numpy().copy() for t in ctx.energy_grad(x, prec))
    for s, e in zip(systems, e0):
        e_ref, _ = oracle.energy_grad(s, s["x"])
        assert abs(e - e_ref) <= (1e-11 if prec == "fp64" else 1e-6) * abs(e_ref)
    runs = []
    for _ in range(3):
        for _ in range(20):
            e, g = ctx.energy_grad(x, prec)
            assert np.array_equal(e.cpu().numpy(), e0) and np.array_equal(g.cpu().numpy(), g0)
        y = x.clone()
        res = ctx.minimize(y, "lbfgs", m=4, max_iter=12, precision=prec)
        runs.append((y.cpu().numpy(), res if isinstance(res, list) else [res]))
    ctx.close()
    for y, res in runs[1:]:
        assert np.array_equal(y, runs[0][0]) and res == runs[0][1]
