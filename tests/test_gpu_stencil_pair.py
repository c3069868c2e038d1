"""The last stage of a Lawson2b step and the first of the next in one launch (3D, FP64): a run of
steps against the same steps taken one at a time, which never pair (bit for bit: the two kernels
share their arithmetic), and against the FP64 oracle at the 1e-12 of every FP64 path."""
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


def solve(mm, problems, at_once):
    import torch
    ctx = mm.Context(0)
    ops = [mm.setup_problem(ctx, p) for p in problems]
    us = [torch.from_numpy(np.ascontiguousarray(p.u0)).cuda() for p in problems]
    steps = problems[0].steps
    for k in [steps] if at_once else [1] * steps:
        if len(ops) == 1:
            mm.step(ops[0], us[0], k)
        else:
            mm.lawson_step_batch(ops, us, k)
    out = [u.cpu().numpy() for u in us], [mm.mm_check(op) for op in ops]
    for op in ops:
        op.close()
    ctx.close()
    return out


def problem(n, seed=61, steps=3):
    return synth.smooth_problem(n, seed, tau=1e-3, steps=steps, scheme="l2b", beta=(3.0, -2.0, 1.0),
                                beta_bar=(0.5, -0.25, 0.0), lam=0.9, r=(0.1, 0.7, -0.4, 0.2))


# (blocks of 512 and 1024 threads, one to three points each; rows far shorter than a block's run and longer than a wave; an
# odd last chunk of planes; the last three stay two launches)
@pytest.mark.parametrize("n", [(2, 65, 128), (3, 301, 30), (17, 129, 65), (33, 200, 97), (65, 66, 67), (65, 129, 65),
                               (129, 200, 33), (257, 200, 15), (256, 30, 200), (257, 400, 15), (490, 200, 15),
                               (31, 33, 2), (48, 50, 1)])
def test_run_matches_single_steps_and_oracle(mm, n):
    p = problem(n)
    (got,), st = solve(mm, [p], True)
    (one,), _ = solve(mm, [p], False)
    assert st == [mm.MM_OK]
    assert np.array_equal(got, one)
    ref = S.solve(p)
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))


def test_group_matches_single_steps(mm):
    ps = [problem((40, 40, 40), 70 + i, 4) for i in range(5)]
    got, one = solve(mm, ps, True)[0], solve(mm, ps, False)[0]
    assert all(np.array_equal(a, b) for a, b in zip(got, one))


def test_nonfinite_state_is_flagged(mm):
    p = problem((17, 129, 65))
    p.u0 = p.u0.copy()
    p.u0[10, 4, 3] = np.inf
    assert solve(mm, [p], True)[1] == [mm.MM_EUNSTABLE]


def test_run_after_an_action_on_the_same_operator(mm):
    """An exponential action leaves its unpadded intermediates in the operator's scratch, also where
    the stage vectors have their row padding."""
    import torch
    p = problem((129, 200, 33))
    (ref,), _ = solve(mm, [p], True)
    ctx = mm.Context(0)
    op = mm.setup_problem(ctx, p)
    u = torch.from_numpy(np.ascontiguousarray(p.u0)).cuda()
    mm.mumode_expv(op, torch.full_like(u, 7.0), torch.empty_like(u))
    mm.step(op, u, p.steps)
    assert np.array_equal(u.cpu().numpy(), ref)
    op.close()
    ctx.close()
