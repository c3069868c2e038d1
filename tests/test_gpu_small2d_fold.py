"""Small 2D solves in one workgroup with folded products (centrosymmetric axes) against the
FP64 oracle and against the plain products of the same kernel; alone and grouped with a
problem that does not fold.

Bounds: a step sums at most 64 + 64 products of magnitude <= max|u| per value, so either form
is within (128 + 20) 2^-53 < 2e-14 of exact per step and vector; 7 steps of two vectors, two
forms: 2 * 7 * 2e-14 < 3e-13 relative to max|u|. The oracle's bar is 1e-12, as elsewhere.
"""
import numpy as np
import pytest

import synth
from oracle import schemes as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_15861_amd as m
    return m


def solve(mm, problems, fold):
    import torch
    ctx = mm.Context(0)
    ctx.set_fold(fold)
    ops = [mm.setup_problem(ctx, p) for p in problems]
    us = [torch.from_numpy(np.ascontiguousarray(p.u0)).cuda() for p in problems]
    if len(ops) == 1:
        mm.step(ops[0], us[0], problems[0].steps)
    else:
        mm.lawson_step_batch(ops, us, problems[0].steps)
    assert all(mm.mm_check(op) == mm.MM_OK for op in ops)
    out = [u.cpu().numpy() for u in us]
    for op in ops:
        op.close()
    ctx.close()
    return out


def problem(n, scheme, beta_bar=(0.0, 0.0)):
    return synth.smooth_problem(n, 47, tau=1e-3, steps=7, scheme=scheme, beta=(3.0, -2.0), beta_bar=beta_bar, lam=0.9,
                                r=(0.1, 0.7, -0.4, 0.2))


@pytest.mark.parametrize("scheme", ["le", "l2b"])
@pytest.mark.parametrize("n", [(1, 1), (1, 64), (2, 1), (2, 3), (15, 16), (17, 32), (33, 31), (34, 64), (63, 63), (64, 63),
                               (64, 64)])
def test_folded_matches_plain_and_oracle(mm, scheme, n):
    p = problem(n, scheme)
    folded, plain, ref = solve(mm, [p], 1)[0], solve(mm, [p], 0)[0], S.solve(p)
    scale = np.max(np.abs(ref))
    assert np.max(np.abs(folded - ref)) <= 1e-12 * scale
    assert np.max(np.abs(folded - plain)) <= 3e-13 * scale


@pytest.mark.parametrize("scheme", ["le", "l2b"])
def test_group_of_both_forms(mm, scheme):
    ps = [problem((63, 40), scheme), problem((63, 40), scheme, (0.5, -0.25))]
    for p, got in zip(ps, solve(mm, ps, 1)):
        assert np.array_equal(got, solve(mm, [p], 1)[0])
