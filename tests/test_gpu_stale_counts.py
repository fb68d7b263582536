"""A context whose finalize or accept count does not stand at zero (calls that
overlapped on it, which its users must not make, can leave one behind)
evaluates and minimizes as a fresh one."""
import os
import subprocess

import numpy as np
import pytest
import torch

import paper_1810_03358_amd as ff
from tests.systems import torsion_chain

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def offsets(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("hostsim") / "offsets")
    sim = os.path.join(ROOT, "tests", "hostsim")
    subprocess.run(["g++", "-std=c++17", "-w", "-pthread", "-I", sim,
                    "-I", os.path.join(ROOT, "paper_1810_03358_amd", "csrc"), os.path.join(sim, "offsets.cpp"),
                    "-o", exe], check=True)
    return [int(v) for v in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]


@pytest.mark.parametrize("sizes", [(300,), (1500,), (5, 700, 64)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_counts_left_behind_do_not_matter(offsets, sizes, prec):
    systems = [torsion_chain(n, 60 + k) for k, n in enumerate(sizes)]
    x = torch.tensor(np.concatenate([np.asarray(s["x"]).reshape(-1, 3) for s in systems]), dtype=torch.float64,
                     device="cuda")
    print(sizes, prec, flush=True)
    # stored in every control block, which is found again by its bytes (no other
    # case's, which the allocator may hand out again)
    tol = 1e-30 * (sum(sizes) + (1 / 3 if prec == "fp32" else 1 / 7))
    ctx = ff.Context(systems, m_max=4)
    e0, g0 = ctx.energy_grad(x, prec)

    def minimize():
        y = x.clone()
        return y, ctx.minimize(y, "lbfgs", m=4, max_iter=8, precision=prec, tol=tol)

    y0, r0 = minimize()
    at = torch.nonzero(ctx.workspace[ctx._ws_ptr - ctx.workspace.data_ptr():][:ctx.workspace.numel() // 8 * 8 - 256]
                       .view(torch.int64) == int(np.array(tol).view(np.int64))).flatten() * 8
    assert len(at) == len(sizes)

    def leave(which):
        torch.cuda.synchronize()
        for a in at.tolist():
            start = ctx._ws_ptr - ctx.workspace.data_ptr() + a + offsets[which]
            ctx.workspace[start:start + 4].view(torch.int32).fill_(1)
        torch.cuda.synchronize()

    for _ in range(2):
        leave(0)
        e = torch.full_like(e0, np.nan)
        g = torch.full_like(g0, np.nan)
        ctx.energy_grad(x, prec, out_e=e, out_g=g)
        assert torch.equal(e, e0) and torch.equal(g, g0)
    for which in (0, 1):
        leave(which)
        y, r = minimize()
        assert torch.equal(y, y0) and r == r0
    ctx.close()
