"""The plan of a whole call can be asked for (CPU only).

hybrid_call_info reports what reconstruct_hybrid runs, hybrid_plan_info what
the steps and the adjoint run; the autotuner tells its candidates apart by the
first and can time the vector kernels where the default is the window form.
"""
import math
import os
from dataclasses import replace

import pytest

import workloads as W

pr = pytest.importorskip("paper_2109_02842_amd")

if not os.path.exists(pr.LIB_PATH):
    pytest.skip("libpolyrecon.so not built", allow_module_level=True)

FINE = W.ImageGrid(nx=70, ny=61, x0=-0.1, y0=-0.09, dx=0.0026, dy=0.003)


@pytest.mark.parametrize("precision,mbp,window", [("fp32", 0, True), ("fp32", -1, False), ("bf16", 0, True),
                                                  ("bf16", 1, True), ("fp16", 1, True), ("fp16", 2, False),
                                                  ("bf16", -1, False)])
def test_call_plan(precision, mbp, window):
    g = pr.make_geometry(W.C2.array)
    opts = dict(precision=precision, mfma_backprojection=mbp)
    call, steps = (f(g, FINE, **opts) for f in (pr.hybrid_call_info, pr.hybrid_plan_info))
    assert call.workspace_bytes == steps.workspace_bytes == pr.hybrid_workspace_bytes(g, FINE, **opts)
    if not window:
        assert call == steps and call.bp_kernel != "window"
        return
    assert call.bp_kernel == "window" and not call.mfma_backprojection and steps.bp_kernel != "window"
    assert call.tile == (16, 16) and call.waves == 8 and call.block == 32
    bins = (W.C2.array.n_scan + 1) // 2             # beside their mirrors
    assert call.n_blocks == -(-bins // 32) == len(call.k_ref)
    assert call.n_fine % 64 == 0 and call.n_fine >= 1.25 * call.n_l
    # a 4x4 pixel group's ranges span 3.4 to 5.66 samples, the step is coarser than the B-spline's
    span = 2 * 3 * math.hypot(FINE.dx, FINE.dy) / call.du
    assert 3.39 < span < 5.67 and call.du > steps.du and call.n_l < steps.n_l


def test_a_requested_kernel_and_small_images_keep_one_plan():
    g = pr.make_geometry(W.C2.array)
    for opts in (dict(kz_block=32), dict(kz_block=64), dict(waves=8), dict(interp="lagrange4"),
                 dict(range_method="resample"), dict(ref_mode="min-k")):
        assert pr.hybrid_call_info(g, FINE, **opts) == pr.hybrid_plan_info(g, FINE, **opts)
    small = pr.make_geometry(W.C1.array)
    assert pr.hybrid_call_info(small, W.C1.grid) == pr.hybrid_plan_info(small, W.C1.grid)


def test_call_plan_errors():
    g = pr.make_geometry(W.C1.array)
    for bad in (dict(l_oversample=1.0), dict(nufft_tol=1.0), dict(tile=3)):
        with pytest.raises(pr.PolyreconError):
            pr.hybrid_call_info(g, W.C1.grid, **bad)
    assert pr.lib().hybrid_call_info(None, None, None, None, None) == pr.PL_EINVAL


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_autotune_tells_the_window_form_from_the_vector_kernels(precision):
    from paper_2109_02842_amd import autotune as at
    g = pr.make_geometry(W.C2.array)
    plans = [pr.hybrid_call_info(g, FINE, **o) for o in at.candidates(g, FINE, precision)]
    shapes = [(p.bp_kernel, p.tile, p.block, p.waves) for p in plans]
    assert len(set(shapes)) == len(shapes)
    assert ("window", (16, 16), 32, 8) in shapes
    assert ("pixel-lanes", (8, 8), 32, 4) in shapes and ("pixel-lanes", (8, 8), 64, 4) in shapes
