"""Roofline figures that bench.py derives from recorded launches (no GPU): the peak that a fused
launch is priced against, and the bytes of Lawson2b stage launches that hold one or two passes."""
import pytest

import bench
import synth


def kernels(**kw):
    out = {k: {"launches": 0, "total_ms": 0.0, "avg_us": 0.0, "work": 0.0}
           for k in ("gemm_k", "gemm_n", "stencil", "fused")}
    for name, (launches, ms, work) in kw.items():
        out[name] = {"launches": launches, "total_ms": ms, "avg_us": 1e3 * ms / launches, "work": work}
    return out


@pytest.mark.parametrize("prob,share", [(lambda: synth.smooth_problem((20, 20), 1, scheme="le"), 1 / 256),
                                        (lambda: synth.paper3d_problem(12, -0.01, 0.53, scheme="sl2"), 1.0),
                                        (lambda: synth.paper2d_problem(16, 0.57, scheme="sl2"), 1.0)])
def test_fused_peak(prob, share):
    roof, name = bench.roofline(kernels(fused=(4, 2.0, 1e9)), "fp64", prob())
    assert name == "fused"
    assert roof["peak"] == pytest.approx(bench.PEAK["fp64"] * share / 1e12)
    assert roof["frac"] == pytest.approx(1e9 / 2e-3 / (bench.PEAK["fp64"] * share))
    assert ("scope" in roof) == (share < 1)


@pytest.mark.parametrize("launches,bytes_per_dof", [(20, 20 * 32), (11, 9 * 40 + 2 * 32)])
def test_stencil_bytes(launches, bytes_per_dof):
    """Ten Lawson2b steps: twenty passes, as twenty launches or with nine pairs."""
    p = synth.smooth_problem((8, 9, 10), 1, scheme="l2b")
    roof, name = bench.roofline(kernels(stencil=(launches, 1.0, 20.0 * p.dof)), "fp64", p)
    assert name == "stencil"
    assert roof["achieved"] == pytest.approx(bytes_per_dof * p.dof / 1e-3 / 1e9)
