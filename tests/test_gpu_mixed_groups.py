"""Groups whose operators share a class (grid, precision, scheme) but not their form: flux and
non-divergence diffusion, Dirichlet and Neumann faces, with and without advection in A. Every
problem of such a group gives the bits of lawson_step on it alone, whatever its neighbours and
their order, in lawson_step_batch and in the request server.

Sizes: axes below and above the first folded length (17), grids whose Lawson2b stages run in
pairs (96^3), 2D grids of the one-workgroup solver (which has the flux form with Dirichlet ends
only) and beyond it."""
import dataclasses
import time

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


ALL = ("plain", "nondiv", "neumann", "advected", "plain")


def forms(n, kinds, scheme="l2b", steps=3, tau=1e-4):
    """Problems of one class: plain ones, non-divergence form, Neumann at x_2 = 1, advection along
    x_1 in A."""
    d = len(n)
    change = {"plain": {}, "nondiv": {"form": "nondiv"}, "neumann": {"bc": (0, 1, 0)[:d]},
              "advected": {"beta_bar": (3.0, 0.0, 0.0)[:d]}}
    return [dataclasses.replace(synth.smooth_problem(n, 300 + i, tau=tau * (1 + 0.3 * i), steps=steps, scheme=scheme,
                                                     beta=(3.0, -2.0, 1.0)[:d]), **change[k])
            for i, k in enumerate(kinds)]


def run(mm, probs, steps):
    import torch
    ctx = mm.Context(0)
    try:
        ops = [mm.setup_problem(ctx, p) for p in probs]
        us = [torch.from_numpy(np.ascontiguousarray(p.u0)).cuda() for p in probs]
        mm.lawson_step_batch(ops, us, steps)
        alone = []
        for op, p in zip(ops, probs):
            u = torch.from_numpy(np.ascontiguousarray(p.u0)).cuda()
            mm.lawson_step(op, u, steps)
            assert mm.mm_check(op) == mm.MM_OK
            alone.append(u.cpu().numpy())
        return [u.cpu().numpy() for u in us], alone
    finally:
        ctx.close()


@pytest.mark.parametrize("n,scheme,kinds", [((16, 12, 9), "l2b", ALL),
                                            ((20, 18, 16), "l2b", ("plain", "nondiv", "plain")),
                                            ((96, 96, 96), "l2b", ("plain", "nondiv")),
                                            ((33, 34, 35), "l2b", ALL), ((40, 5, 63), "le", ALL),
                                            ((17, 16, 70), "l2b", ALL),
                                            ((90, 70), "l2b", ALL), ((130, 70), "le", ALL),
                                            ((129, 130, 40), "l2b", ("advected", "plain")),
                                            ((40, 33), "l2b", ALL), ((63, 16), "le", ALL),
                                            ((64, 5), "l2b", ("plain", "neumann"))])
@pytest.mark.parametrize("reverse", [False, True])
def test_mixed_group_equals_alone(mm, n, scheme, kinds, reverse):
    probs = forms(n, kinds[::-1] if reverse else kinds, scheme)
    print(f"[mixed] {n} {scheme} {kinds} reverse={reverse}", flush=True)
    grouped, alone = run(mm, probs, 3)
    for g, a in zip(grouped, alone):
        assert np.isfinite(a).all()
        assert np.array_equal(g, a)


def serve(mm, batch):
    srv = mm.Server(0, max_active=8)
    try:
        ids = [mm.solve_submit(srv, p)[1] for p in batch]
        out = []
        for i, p in zip(ids, batch):
            t0 = time.time()
            while (r := mm.solve_poll(srv, i, p.shape))[0] == mm.MM_NOT_READY:
                assert time.time() - t0 < 60
                time.sleep(0.001)
            out.append(r)
        return out, srv.counters()
    finally:
        srv.close()


@pytest.mark.parametrize("kinds", [("plain", "nondiv", "nondiv", "plain"), ALL])
def test_server_mixes_forms(mm, kinds):
    """Requests of one class and different forms, long enough to be advanced together: each equals
    the same request served alone."""
    probs = [dataclasses.replace(p, steps=600) for p in forms((33, 20, 24), kinds, tau=1e-5)]
    together, counters = serve(mm, probs)
    assert counters["mean_group"] > 1.0
    for p, (st, u, _) in zip(probs, together):
        assert st == mm.MM_OK
        assert np.array_equal(u, serve(mm, [p])[0][0][1])
