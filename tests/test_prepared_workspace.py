"""A prepared workspace keeps its tables through the adjoint and the steps.

A prepared call of a plan that takes the window form reads its own tables; the
adjoint and the steps with the same arguments write the vector plan's.  Both
lie in one workspace, so the first must be past the second: the workspace
holds the vector plan's and the window form's tables beside it.
"""
import os
from dataclasses import replace

import pytest

import workloads as W

torch = pytest.importorskip("torch")
pr = pytest.importorskip("paper_2109_02842_amd")

if not os.path.exists(pr.LIB_PATH):
    pytest.skip("libpolyrecon.so not built", allow_module_level=True)

ARRAY = replace(W.C1.array, n_scan=229, n_elem=9, n_freq=20)
GRID = W.ImageGrid(nx=45, ny=29, x0=-0.053, y0=-0.039, dx=0.0026, dy=0.0026)


def test_window_tables_lie_past_the_vector_plan():
    g = pr.make_geometry(ARRAY)
    tiles, blocks = 3 * 2, 4
    tables = tiles * g.n_channels * (48 + 8 * blocks) + 12 * ARRAY.n_scan * ARRAY.n_freq
    vector = pr.hybrid_workspace_bytes(g, GRID, mfma_backprojection=-1)
    assert pr.hybrid_workspace_bytes(g, GRID) >= vector + tables
    # a kernel asked for: one plan, no second tables
    assert pr.hybrid_workspace_bytes(g, GRID, kz_block=32) == vector


@pytest.mark.gpu
def test_prepared_calls_between_adjoints_and_steps():
    g = pr.make_geometry(ARRAY)
    gen = torch.Generator(device="cuda").manual_seed(1)
    echo = torch.view_as_complex(torch.randn(*g.echo_shape, 2, device="cuda", generator=gen))
    want = pr.reconstruct_hybrid(g, GRID, echo)
    assert not torch.equal(want, pr.reconstruct_hybrid(g, GRID, echo, mfma_backprojection=-1))
    adj = pr.adjoint_hybrid(g, GRID, want)
    ws = pr.hybrid_prepare(g, GRID)
    for _ in range(2):
        assert torch.equal(pr.reconstruct_hybrid(g, GRID, echo, ws=ws, prepared=True), want)
        assert torch.equal(pr.adjoint_hybrid(g, GRID, want, ws=ws), adj)
        spec = pr.scan_fft(g, echo, ws=ws)
        q, _ = pr.range_compress(g, GRID, spec, ws=ws)
        pr.kz_ifft(g, GRID, pr.backproject(g, GRID, q, ws=ws), ws=ws)
    assert torch.equal(pr.reconstruct_hybrid(g, GRID, echo, ws=ws, prepared=True), want)
