"""phi1 actions and ERK steps in the folded sine basis (FP64, zero Dirichlet data and no
advection in A on every axis) against the oracle and against the plain products: axes of
one, two and three points, odd and even lengths (a middle coefficient or none), axes of
either folded kernel, 2D and 3D, exact phi1 and quadratures of one and several nodes.
"""
import numpy as np
import pytest

import synth
from oracle import adr, expo

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-12


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_15861_amd as m
    return m


@pytest.mark.parametrize("q", [0, 1, 6])
@pytest.mark.parametrize("n", [(1, 1), (2, 3), (40, 33), (1, 2, 3), (16, 17, 2), (35, 21, 18), (9, 300, 32), (257, 3, 20),
                               (511, 33), (40, 512), (385, 6, 450)])
def test_phi1_action(mm, n, q):
    import torch
    p = synth.smooth_problem(n, 61, tau=2e-3, scheme="etd2rk", q=q)
    V = np.random.default_rng(62).standard_normal(p.shape)
    ctx = mm.Context(0)
    op = mm.setup_problem(ctx, p)
    out = torch.full(p.shape, float("nan"), dtype=torch.float64, device="cuda")
    mm.mumode_phi1v(op, torch.from_numpy(V).cuda(), out)
    got = out.cpu().numpy()
    op.close()
    ctx.close()
    o = expo.KronOperator(p.n, adr.extracted_amax(p.a), p.lam, p.beta_bar, p.tau)
    ref = o.phi1v_quad(V, q) if q else o.phi1v_exact(V)
    assert np.max(np.abs(got - ref)) <= FP64_TOL * np.max(np.abs(ref))


@pytest.mark.parametrize("scheme,q", [("etd2rk", 0), ("etd2rk", 4), ("erk2p1f", 0), ("erk2p1f", 3), ("erk2p2", 0), ("ee", 0)])
def test_steps_against_plain_products(mm, scheme, q):
    import torch
    p = synth.smooth_problem((33, 18, 31), 63, tau=1e-3, scheme=scheme, q=q)
    got = {}
    for mode in (0, 1):
        ctx = mm.Context(0)
        ctx.set_fold(mode)
        op = mm.setup_problem(ctx, p)
        u = torch.from_numpy(p.u0).cuda()
        mm.step(op, u, 3)
        got[mode] = u.cpu().numpy()
        op.close()
        ctx.close()
    assert np.max(np.abs(got[1] - got[0])) <= FP64_TOL * np.max(np.abs(got[0]))
