"""Folded FP64 mode products with the factor held in registers, at the edges of their shapes.

Each triple puts one short axis against two long ones, so that the short axis's product (its
length decides the kernel: row tiles of 16 folded positions, 17 <= n <= 256) walks over several
tiles per workgroup, on odd unpadded rows (the last column pair starts one column back),
ragged units of 16 fibers and middle positions in every place of a row tile; the long axes
run the widest workgroups. The results must meet the FP64 bar of the exponential action
against the oracle; the tolerance is that of the folded products' other tests.
"""
import numpy as np
import pytest

import synth
from oracle import adr, expo

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-12

SHAPES = [(17, 253, 203), (203, 18, 253), (253, 203, 17), (201, 255, 16), (49, 251, 201), (201, 34, 251),
          (255, 201, 33), (65, 199, 251), (207, 64, 255), (255, 241, 66), (81, 223, 249), (225, 97, 211),
          (256, 161, 130), (145, 256, 177), (209, 193, 240)]


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_15861_amd as m
    return m


@pytest.mark.parametrize("n", SHAPES)
def test_exp_action(mm, n):
    import torch
    p = synth.smooth_problem(n, 51, tau=1e-3)
    V = np.random.default_rng(52).standard_normal(p.shape)
    ctx = mm.Context(0)
    op = mm.setup_problem(ctx, p)
    out = torch.full(p.shape, float("nan"), dtype=torch.float64, device="cuda")
    mm.mumode_expv(op, torch.from_numpy(V).cuda(), out)
    got = out.cpu().numpy()
    op.close()
    ctx.close()
    ref = expo.KronOperator(p.n, adr.extracted_amax(p.a), p.lam, p.beta_bar, p.tau).expv(1.0, V)
    assert np.max(np.abs(got - ref)) <= FP64_TOL * np.max(np.abs(ref))


@pytest.mark.parametrize("n", [(33, 251, 64), (255, 66, 130)])
def test_scaled_and_added_output(mm, n):
    """alpha and the added term (u+ = u + tau e^{tau A} F(u), the scheme that uses both) against
    the plain products."""
    import torch
    p = synth.smooth_problem(n, 53, tau=1e-4, scheme="sle")
    u0 = np.random.default_rng(54).standard_normal(p.shape)
    got = {}
    for mode in (0, 1):
        ctx = mm.Context(0)
        ctx.set_fold(mode)
        op = mm.setup_problem(ctx, p)
        u = torch.from_numpy(u0).cuda()
        mm.step(op, u, 2)
        got[mode] = u.cpu().numpy()
        op.close()
        ctx.close()
    # both sum in FP64: a few units of rounding per sum of n terms, over two steps
    assert np.max(np.abs(got[1] - got[0])) <= 1e-12 * np.max(np.abs(got[0]))


@pytest.mark.parametrize("n", [(511, 300), (383, 449), (257, 512)])
def test_wide_factors_in_lawson_steps(mm, n):
    """axes of 257 to 512 points on grids of few tiles (one wave per SIMD, row groups), in the
    padded layout of the Lawson steps, against the plain products."""
    import torch
    p = synth.smooth_problem(n, 55, tau=1e-4, scheme="l2b", beta=(0.5, 0.5))
    got = {}
    for mode in (0, 1):
        ctx = mm.Context(0)
        ctx.set_fold(mode)
        op = mm.setup_problem(ctx, p)
        u = torch.from_numpy(p.u0).cuda()
        mm.step(op, u, 2)
        got[mode] = u.cpu().numpy()
        op.close()
        ctx.close()
    # the last stage adds tau/2 g(U): differences of U grow by 1 + 2 d tau (a_max - a_min)/h^2
    grow = 1.0 + 4 * 1e-4 * 1.8 * (max(n) + 1) ** 2
    assert np.max(np.abs(got[1] - got[0])) <= 2 * grow * 1e-13 * np.max(np.abs(got[0]))
