"""Which ERK operators run in the folded sine basis: those whose steps are estimated faster there
than with one product per node (few nodes and small grids are not). The number of product
launches of a step tells the route; either agrees with the plain products (fold mode 0) to
FP64 rounding."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-12


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_15861_amd as m
    return m


CASES = [((16, 16, 16), "etd2rk", 7, False), ((31, 31, 31), "etd2rk", 4, False),
         ((63, 63, 63), "etd2rk", 2, False), ((127, 127, 127), "etd2rk", 1, False),
         ((127, 127, 127), "erk2p1f", 1, False), ((100, 100, 20), "etd2rk", 4, False),
         ((255, 255), "etd2rk", 2, False), ((31, 31, 31), "etd2rk", 0, False), ((160, 160), "erk2p1f", 0, False),
         ((12, 12, 12), "ee", 0, False), ((16, 9, 12), "erk2p2", 0, False),
         ((127, 127, 127), "etd2rk", 4, True), ((110, 110, 110), "erk2p1f", 4, True),
         ((64, 31, 256), "etd2rk", 6, True), ((511, 511), "etd2rk", 4, True), ((12, 13, 300), "etd2rk", 7, True),
         ((80, 80, 80), "etd2rk", 0, True), ((96, 97, 81), "erk2p2", 0, True), ((383, 300), "ee", 0, True)]


@pytest.mark.parametrize("n,scheme,q,sine", CASES)
def test_route(mm, n, scheme, q, sine):
    import torch
    # (A = 0.5 L less the a_min..a_max part: a constant, so that no stage multiplies rounding)
    p = synth.constant_problem(n, 65, a_const=0.5, tau=1e-4, scheme=scheme, q=q, beta=(0.1,) * len(n), r=synth.R_CUBIC)
    got, launches = {}, {}
    for mode in (0, 1):
        ctx = mm.Context(0)
        ctx.set_fold(mode)
        op = mm.setup_problem(ctx, p)
        u = torch.from_numpy(p.u0).cuda()
        ctx.timing(True)
        mm.step(op, u, 1)
        launches[mode] = sum(ctx.timing_read(k)[0] for k in (mm.MM_KIND_GEMM_K, mm.MM_KIND_GEMM_N))
        got[mode] = u.cpu().numpy()
        ctx.close()
    d, stages = len(n), 1 if scheme == "ee" else 2
    # a transform and its inverse per stage (with exact functions also without the basis), or one
    # grouped action
    assert launches[0] == stages * d * (1 if q else 2)
    assert launches[1] == stages * d * (2 if sine or not q else 1)
    if q == 0:
        # the exact forms differ in their bits only where the route differs
        assert np.array_equal(got[0], got[1]) == (not sine)
    assert np.max(np.abs(got[1] - got[0])) <= FP64_TOL * np.max(np.abs(got[0]))


def test_plain_form_is_built_on_demand(mm):
    """Fold mode 0 gives operators in the sine basis their node products, those set up before it and
    under it alike: the same bits of phi1 actions and steps. A graph recorded before keeps its
    results."""
    import torch
    n, q = (97, 96, 98), 7
    p = synth.constant_problem(n, 66, a_const=0.5, tau=1e-4, scheme="etd2rk", q=q, beta=(0.1,) * 3, r=synth.R_CUBIC)

    def results(op):
        u = torch.from_numpy(p.u0).cuda()
        out = torch.empty_like(u)
        mm.mumode_phi1v(op, u, out)
        mm.step(op, u, 2)
        return u.cpu().numpy(), out.cpu().numpy()

    late, early = mm.Context(0), mm.Context(0)
    early.set_fold(0)
    op = mm.setup_problem(late, p)
    sine = results(op)
    g, u = torch.cuda.CUDAGraph(), torch.from_numpy(p.u0).cuda()
    with torch.cuda.graph(g):
        mm.step(op, u, 2)
    late.set_fold(0)
    plain = results(op)
    ref = results(mm.setup_problem(early, p))
    for a, b, c in zip(plain, ref, sine):
        assert np.array_equal(a, b)
        assert np.max(np.abs(a - c)) <= FP64_TOL * np.max(np.abs(c))
    late.set_fold(1)
    again = results(op)
    assert np.array_equal(again[0], sine[0]) and np.array_equal(again[1], sine[1])
    for _ in range(3):
        u.copy_(torch.from_numpy(p.u0))
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(u.cpu().numpy(), sine[0])
    op.close()
    late.set_fold(0)
    late.close()
    early.close()


def test_plain_form_is_built_while_a_graph_is_recorded(mm):
    """Fold mode 0 set between two steps of a recorded graph: the first replays in the sine basis, the
    second by nodes, as the same calls do directly."""
    import torch
    p = synth.constant_problem((97, 96, 98), 68, a_const=0.5, tau=1e-4, scheme="etd2rk", q=7, beta=(0.1,) * 3)
    results = []
    for record in (False, True):
        ctx = mm.Context(0)
        op = mm.setup_problem(ctx, p)
        u = torch.from_numpy(p.u0).cuda()

        def steps():
            mm.step(op, u, 1)
            ctx.set_fold(0)
            mm.step(op, u, 1)

        if record:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                steps()
            for _ in range(2):
                u.copy_(torch.from_numpy(p.u0))
                g.replay()
                torch.cuda.synchronize()
                results.append(u.cpu().numpy())
        else:
            steps()
            results.append(u.cpu().numpy())
        ctx.close()
    assert all(np.array_equal(r, results[0]) for r in results)


def test_memory_of_an_operator_in_the_sine_basis():
    """It holds seven grid functions and the coefficient, not the scratch of the node products
    (2 (q + 1) grid functions) as well: free memory around a setup, in a process of its own (freed
    memory stays in the device's pool)."""
    import os
    import subprocess
    import sys
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    code = """
import torch, synth, paper_2303_15861_amd as mm
n = (130, 131, 132)
p = synth.constant_problem(n, 67, a_const=0.5, tau=1e-4, scheme="etd2rk", q=7, beta=(0.1,) * 3)
ctx = mm.Context(0)
free = torch.cuda.mem_get_info()[0]
op = mm.setup_problem(ctx, p)
torch.cuda.synchronize()
print((free - torch.cuda.mem_get_info()[0]) / (8 * n[0] * n[1] * n[2]))
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    # (also in it: the operator's factors and the test's own copy of the coefficient; with the
    # node products' scratch it is above 22)
    assert float(r.stdout.split()[-1]) < 14
