"""Exponential actions give the same bits whichever way their plain products are launched: as one
launch per x3 slab, as separate tiled products (a product tile set by the caller keeps them) and
through mumode_expv_noalloc. Grids with n1, n2 <= 64 (slab launch) down to a single point along x3,
the largest cubes that mumode_expv_noalloc takes, and larger products with folding off; where such
products fold (192 tiles of 128 fibers x 64 folded positions on) the two agree to rounding: sums of n1 + n2 + n3
products with row sums <= 1 on either side, 2 (n1 + n2 + n3 + 30) 2^-53 max |u| < 2e-13."""
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


def actions(mm, n, fold, tiles=(0, 32, 64)):
    import torch
    p = synth.smooth_problem(n, 73, tau=1e-3, steps=1, scheme="l2b")
    x = torch.from_numpy(np.ascontiguousarray(p.u0)).cuda()
    outs = []
    for tile in tiles:
        ctx = mm.Context(0)
        ctx.set_gemm_tile(tile)
        ctx.set_fold(fold)
        op = mm.setup_problem(ctx, p)
        out = torch.full_like(x, float("nan"))
        mm.mumode_expv(op, x, out)
        factors = [torch.from_numpy(np.ascontiguousarray(op.factor(mu, 0))).cuda() for mu in range(len(n))]
        outs.append(out.cpu().numpy())
        out.fill_(float("nan"))
        mm.mumode_expv_noalloc(ctx, factors, x, out)
        outs.append(out.cpu().numpy())
        op.close()
        ctx.close()
    return outs


@pytest.mark.parametrize("n", [(2, 2, 2), (2, 64, 1), (15, 17, 3), (31, 31, 31), (33, 16, 40), (64, 63, 20),
                               (64, 64, 64), (48, 5, 180)])
def test_slab_action_bits(mm, n):
    outs = actions(mm, n, 1)
    assert all(np.array_equal(o, outs[0]) for o in outs)


@pytest.mark.parametrize("n", [(100, 100, 200), (127, 127, 130), (64, 64, 300), (61, 70, 45), (300, 20)])
def test_plain_action_bits(mm, n):
    outs = actions(mm, n, 0)
    assert all(np.array_equal(o, outs[0]) for o in outs)


@pytest.mark.parametrize("n", [(127, 127, 127), (128, 128, 128)])
def test_largest_cubes_bits(mm, n):
    outs = actions(mm, n, 1, tiles=(0, 64))
    assert all(np.array_equal(o, outs[0]) for o in outs)


@pytest.mark.parametrize("n,fold", [((100, 100, 200), 1), ((127, 127, 130), 1), ((31, 31, 31), 2)])
def test_folded_action_agrees(mm, n, fold):
    outs = actions(mm, n, fold, tiles=(0,))
    assert not np.array_equal(outs[0], outs[1])
    assert np.max(np.abs(outs[0] - outs[1])) <= 2e-13
