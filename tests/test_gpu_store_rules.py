"""Register-held products on both sides of the limits up to which their outputs go through the
caches: small outputs that a tiled product reads next (6 MiB), and outputs in rows of partial
128-byte lines (16 MiB), against the plain products of fold mode 0.

Bound: sums of n1 + n2 + n3 <= 4300 products with row sums <= 1 in either form, one action:
2 (4300 + 30) 2^-53 max|u| < 1e-12."""
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


@pytest.mark.parametrize("n", [(65, 1500), (190, 4000), (200, 4000), (33, 34, 700),            # a tiled product is next
                               (127, 129, 127), (129, 129, 129), (143, 40, 400), (144, 40, 400)])   # rows and lines
def test_action(mm, n):
    import torch
    p = synth.constant_problem(n, 95, a_const=1.0, tau=1e-5, scheme="l2b")
    V = torch.from_numpy(np.random.default_rng(96).uniform(-1, 1, p.shape)).cuda()
    out = {}
    for mode in (0, 2):
        ctx = mm.Context(0)
        ctx.set_fold(mode)
        op = mm.setup_problem(ctx, p)
        got = torch.full_like(V, float("nan"))
        mm.mumode_expv(op, V, got)
        out[mode] = got.cpu().numpy()
        ctx.close()
    assert np.max(np.abs(out[2] - out[0])) <= 1e-12
