"""Lawson steps of small periodic 2D problems as launches of product tasks (FP64, flux form, axes
of 2 to 256 points) against the FFT oracle: every scheme, tile and block edges of both axes
(one to sixteen blocks of 16 points per axis, unequal counts), with a velocity field and with
constant velocities. Axes of 257 points take the separate passes and must agree as well."""
import numpy as np
import pytest

from oracle import spectral
from test_gpu_spectral import random_periodic

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-12


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_15861_amd as m
    return m


@pytest.mark.parametrize("scheme", ["le", "l2b", "sle", "l2a", "sl2"])
@pytest.mark.parametrize("n,velocity", [((2, 3), True), ((16, 17), False), ((15, 33), True), ((64, 48), True),
                                        ((129, 5), False), ((255, 31), True), ((6, 256), True), ((257, 8), True)])
def test_steps_match_oracle(mm, scheme, n, velocity):
    import torch
    p = random_periodic(n, 81, velocity=velocity, scheme=scheme, steps=3, tau=1e-4)
    ctx = mm.Context(0)
    op = mm.setup_problem(ctx, p)
    u = torch.from_numpy(np.ascontiguousarray(p.u0)).cuda()
    mm.step(op, u, p.steps)
    assert mm.mm_check(op) == mm.MM_OK
    got = u.cpu().numpy()
    op.close()
    ctx.close()
    ref = spectral.solve(p)
    assert np.max(np.abs(got - ref)) <= FP64_TOL * np.max(np.abs(ref))
