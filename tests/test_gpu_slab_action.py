"""Exponential actions on grids with n1, n2 <= 64, whose products along x1 and x2 are one launch
per x3 slab: against the separate products (a product tile set by the caller keeps them), against
mumode_expv_noalloc and against the FP64 oracle.

Bounds: three contractions of at most 64 + 64 + n3 products of factors with row sums <= 1, either
form within (n1 + n2 + n3 + 30) 2^-53 max|u| of exact; twice that between two forms, <= 1e-13 at
n3 <= 300."""
import numpy as np
import pytest

import synth
from oracle import adr, expo

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_15861_amd as m
    return m


@pytest.mark.parametrize("n", [(2, 2, 2), (2, 64, 1), (15, 17, 3), (31, 31, 31), (33, 16, 40), (64, 63, 20), (64, 64, 64),
                               (48, 5, 300)])
def test_action_matches_separate_products(mm, n):
    import torch
    p = synth.smooth_problem(n, 71, tau=1e-3, steps=1, scheme="l2b")
    outs = []
    for tile in (0, 32):
        ctx = mm.Context(0)
        ctx.set_gemm_tile(tile)
        op = mm.setup_problem(ctx, p)
        u = torch.from_numpy(np.ascontiguousarray(p.u0)).cuda()
        out = torch.empty_like(u)
        mm.mumode_expv(op, u, out)
        mm.mumode_expv(op, u, u)   # in place
        assert torch.equal(out, u)
        outs.append(out.cpu().numpy())
        factors = [torch.from_numpy(np.ascontiguousarray(op.factor(mu, 0))).cuda() for mu in range(3)]
        mm.mumode_expv_noalloc(ctx, factors, torch.from_numpy(np.ascontiguousarray(p.u0)).cuda(), out)
        outs.append(out.cpu().numpy())
        op.close()
        ctx.close()
    scale = np.max(np.abs(p.u0))
    assert all(np.max(np.abs(o - outs[0])) <= 1e-13 * scale for o in outs)
    ref = expo.KronOperator(p.n, adr.extracted_amax(p.a), p.lam, p.beta_bar, p.tau).expv(1.0, p.u0)
    assert np.max(np.abs(outs[0] - ref)) <= 1e-12 * np.max(np.abs(ref))
