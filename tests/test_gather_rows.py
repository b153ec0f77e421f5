"""The pixel-per-lane back-projection with split k_z rows (few items) is the
unsplit kernel bit for bit.

A batch always runs the unsplit kernel's code, a single call with at most 256
(k_z block, tile) items the split one, so each case compares the two.  Edges:
channel counts around the eight-channel step, scan lengths around the eight
rows, 32- and 64-bin blocks, both arrays, partial tiles, and the last item
count on either side of the rule.
"""
import os
from dataclasses import replace

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pr = pytest.importorskip("paper_2109_02842_amd")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pr.LIB_PATH):
        pytest.fail("libpolyrecon.so is not built")
    yield
    torch.cuda.synchronize()


MULTI = W.ArrayDesc(mode="multi", n_chords=3, radius=0.5, n_elem=9, spacing=W._D_MULTI, n_tx=2, n_scan=41,
                    scan_step=0.005, n_freq=16, f_start=26e9, f_stop=34e9)


def mono(chords, elem, scan):
    return replace(W.C1.array, n_chords=chords, n_elem=elem, n_scan=scan)


@pytest.mark.parametrize("array,nx,ny,pitch,block", [
    (mono(1, 1, 9), 1, 1, 0.005, 32),
    (mono(1, 7, 24), 9, 13, 0.003, 32),
    (mono(2, 4, 33), 32, 32, 0.009, 32),
    (mono(3, 3, 100), 17, 8, 0.004, 64),
    (mono(1, 17, 7), 45, 29, 0.006, 64),
    (MULTI, 27, 35, 0.004, 32),
    (mono(1, 5, 32), 128, 128, 0.004, 32),     # 256 items
    (mono(1, 5, 32), 129, 128, 0.004, 32),     # 272 items: unsplit on both sides
])
def test_split_rows_are_the_unsplit_kernel(array, nx, ny, pitch, block):
    grid = W.ImageGrid(nx=nx, ny=ny, x0=-pitch * nx / 2, y0=-pitch * ny / 2, dx=pitch, dy=pitch)
    geom = pr.make_geometry(array)
    opts = dict(mfma_backprojection=-1, kz_block=block)
    assert pr.hybrid_plan_info(geom, grid, **opts).bp_kernel == "pixel-lanes"
    print(array.mode, array.n_scan, nx, ny, block, flush=True)
    echo = torch.from_numpy(W.random_echo(array, 8)).cuda()
    single = pr.reconstruct_hybrid(geom, grid, echo, **opts)
    batch = pr.HybridBatch([geom], [grid], [opts])
    assert batch.queued_scans == 1
    assert torch.equal(single, pr.reconstruct_hybrid_batch(batch, [echo])[0])
