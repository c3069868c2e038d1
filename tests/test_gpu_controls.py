"""Steps and actions with fused launches (x3 slabs, small periodic grids) follow the context's
controls: a product tile set by the caller and fold mode 2 keep the separate products."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_15861_amd as m
    return m


def fused_launches(mm, p, tile=0, fold=1, action=False):
    """Result and number of fused launches of two steps (or one action)."""
    import torch
    ctx = mm.Context(0)
    try:
        ctx.set_gemm_tile(tile)
        ctx.set_fold(fold)
        op = mm.setup_problem(ctx, p)
        u = torch.from_numpy(np.ascontiguousarray(p.u0)).cuda()
        ctx.timing(True)
        if action:
            mm.mumode_expv(op, u, u)
        else:
            mm.step(op, u, 2)
        assert mm.mm_check(op) == mm.MM_OK
        n = ctx.timing_read(mm.MM_KIND_FUSED)[0]
        return u.cpu().numpy(), n
    finally:
        ctx.close()


def agree(a, b):
    # (two steps; products and stages of another order of sums: rounding)
    return np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))


@pytest.mark.parametrize("scheme", ["sle", "l2a", "sl2"])
def test_slab_steps(mm, scheme):
    p = synth.smooth_problem((33, 20, 18), 81, tau=1e-3, scheme=scheme, lam=0.6)
    ref, n = fused_launches(mm, p)
    assert n > 0
    for kw in ({"tile": 64}, {"fold": 2}):
        u, n = fused_launches(mm, p, **kw)
        assert n == 0 and agree(u, ref)


@pytest.mark.parametrize("scheme", ["le", "l2b", "sl2"])
def test_periodic_steps(mm, scheme):
    p = synth.paper2d_problem(48, 0.6, scheme=scheme, steps=256)
    ref, n = fused_launches(mm, p)
    assert n > 0
    u, n = fused_launches(mm, p, tile=64)
    assert n == 0 and agree(u, ref)


def test_slab_action(mm):
    p = synth.smooth_problem((33, 20, 18), 82, tau=1e-3)
    ref, n = fused_launches(mm, p, action=True)
    assert n > 0
    for kw in ({"tile": 64}, {"fold": 2}):
        u, n = fused_launches(mm, p, action=True, **kw)
        assert n == 0 and agree(u, ref)
