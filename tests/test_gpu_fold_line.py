"""Where the default fold mode takes the register-held folded kernel: from 129 to 256 points only
from a least number of 16-fiber units on (few units are the plain kernel's), on either axis. The
recorded work of a launch tells which form ran; results agree with the plain products.

Bound: one Lawson2b step, sums of at most 256 + m products with row sums <= 1 in either form, and a
last stage that multiplies their difference by 1 + 2 d tau (a_max - a_min)/h^2 (a constant: 1) and
the advection's tau |beta| / h: 2 (256 + m + 30) 2^-53 (1 + 1e-7 2 m) < 2e-12 at m <= 2900."""
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


# points, fibers of one vector below which the plain product runs (two vectors: the units count twice)
LINES = [(129, 1536), (144, 1536), (160, 2816), (176, 1536), (191, 2816), (224, 1280), (255, 1280)]


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("n,m,folded", [(n, m + d, d >= 0) for n, m in LINES for d in (-16, 0)] +
                         [(128, 17, True), (200, 17, True), (245, 17, True), (257, 33, True)])
def test_least_fibers(mm, axis, n, m, folded):
    import torch
    shape = (n, m) if axis == 0 else (m, n)
    p = synth.constant_problem(shape, 91, a_const=1.0, tau=1e-7, scheme="l2b", beta=(1.0, 1.0), r=synth.R_CUBIC)
    out = {}
    for mode in (0, 1):
        ctx = mm.Context(0)
        ctx.set_fold(mode)
        op = mm.setup_problem(ctx, p)
        u = torch.from_numpy(p.u0).cuda()
        ctx.timing(True)
        mm.step(op, u, 1)
        out[mode] = u.cpu().numpy()
        count, _, work = ctx.timing_read(mm.MM_KIND_GEMM_K if axis == 0 else mm.MM_KIND_GEMM_N)
        assert count == 1
        f = n - n // 2
        assert work == 2 * m * (4 * f * f if mode and folded else 2 * n * n)
        ctx.close()
    assert np.max(np.abs(out[1] - out[0])) <= 2e-12 * np.max(np.abs(out[0]))
