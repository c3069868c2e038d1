"""Steps whose stage vectors and first two products run slab by slab (FP64, n1 and n2 at most
64; the schemes sle, l2a and sl2) against the oracle: tile edges of both axes (2 to 64
points, rows of odd length whose last pair is the grid's last value), single planes, both
diffusion forms, Dirichlet and zero-normal-derivative ends on every axis."""
import numpy as np
import pytest

import synth
from oracle import adr3d

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_15861_amd as m
    return m


def mixed_problem(n, bc, form, seed, **kw):
    p = synth.smooth_problem(n, seed, **kw)
    a = p.a.copy()
    for mu in range(3):
        if bc[mu]:   # the node beyond a zero normal derivative holds the mirror value
            dst, src = [slice(None)] * 3, [slice(None)] * 3
            dst[2 - mu], src[2 - mu] = n[mu] + 1, n[mu] - 1
            a[tuple(dst)] = a[tuple(src)]
    p.a, p.bc, p.form = a, tuple(bc), form
    return p


@pytest.mark.parametrize("scheme", ["sle", "l2a", "sl2"])
@pytest.mark.parametrize("n,bc,form", [((2, 3, 1), (0, 0, 0), "flux"), ((16, 17, 2), (1, 0, 1), "flux"),
                                       ((33, 15, 3), (0, 1, 0), "nondiv"), ((31, 32, 9), (1, 1, 1), "nondiv"),
                                       ((48, 49, 4), (0, 0, 1), "flux"), ((63, 64, 5), (1, 0, 0), "flux"),
                                       ((64, 63, 18), (0, 1, 1), "nondiv"), ((63, 63, 7), (0, 0, 0), "flux")])
def test_steps_match_oracle(mm, scheme, n, bc, form):
    import torch
    p = mixed_problem(n, bc, form, 71, tau=1e-4, steps=3, scheme=scheme, lam=0.6, beta=(3.0, -2.0, 1.5),
                      beta_bar=(1.0, -0.5, 0.25), r=(0.1, 0.7, -0.4, 0.2))
    ctx = mm.Context(0)
    op = mm.setup_problem(ctx, p)
    u = torch.from_numpy(p.u0).cuda()
    mm.step(op, u, p.steps)
    assert mm.mm_check(op) == mm.MM_OK
    got = u.cpu().numpy()
    op.close()
    ctx.close()
    ref = adr3d.solve(p)
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
