"""Full-size reconstructions on the kernels that a default call leaves to the
window form: the pixel-per-lane kernels behind the FP32 NUFFT and the BF16 and
FP16 range compression, the split matrix-core kernel, and the batch queue of
pixel-per-lane scans.  Against sampled (k_z, pixel) pairs of the float64 oracle;
tolerances 1e-4 (FP32) and 1e-3 (BF16, FP16), those of the method's other
full-size checks.
"""
import os

import numpy as np
import pytest

import workloads as W
from oracle import geometry as ogeom
from oracle import hybrid as ohyb

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pr = pytest.importorskip("paper_2109_02842_amd")

VECTOR = dict(mfma_backprojection=-1)
SPLIT = dict(mfma_backprojection=1, tile=16, tile_y=16, kz_block=64)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pr.LIB_PATH):
        pytest.fail("libpolyrecon.so is not built")
    yield
    torch.cuda.synchronize()


def sampled_error(a, grid, echo, img, seed, n_pix):
    """Relative L2 error of the image's spectrum at sampled (k_z, pixel) pairs."""
    assert np.all(np.isfinite(img))
    kap = sorted(set(W.random_subset(a.n_scan, 2, seed).tolist() + [0, a.n_scan // 2]))
    pix = np.unique(np.concatenate([W.random_subset(grid.nx * grid.ny, n_pix, seed + 1), [0, grid.nx * grid.ny - 1]]))
    px, py = ohyb.pixel_grid(grid)
    ref = ohyb.spectrum_at(ogeom.build(a), ohyb.scan_spectrum(echo), kap, px[pix], py[pix])
    got = np.fft.fft(img.astype(np.complex128).reshape(a.n_scan, -1), axis=0)[np.ix_(kap, pix)]
    return float(np.linalg.norm(got - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("wl,precision,opts,kernel", [
    (W.C2, "fp32", VECTOR, "pixel-lanes"), (W.C3, "fp32", VECTOR, "pixel-lanes"),
    (W.C2, "bf16", VECTOR, "pixel-lanes"), (W.C2, "fp16", VECTOR, "pixel-lanes"),
    (W.C3, "bf16", VECTOR, "pixel-lanes"), (W.C2, "bf16", SPLIT, "mfma"), (W.C2, "fp16", SPLIT, "mfma"),
    (W.C3, "bf16", SPLIT, "mfma"),
], ids=["C2-fp32", "C3-fp32", "C2-bf16", "C2-fp16", "C3-bf16", "C2-bf16-split", "C2-fp16-split", "C3-bf16-split"])
def test_full_size_on_an_asked_for_kernel(wl, precision, opts, kernel):
    a, opts = wl.array, dict(opts, precision=precision)
    g = pr.make_geometry(a)
    assert pr.hybrid_call_info(g, wl.grid, **opts).bp_kernel == kernel
    s = W.random_echo(a, 21)
    print("full size", wl.name, opts, flush=True)
    img = pr.reconstruct_hybrid(g, wl.grid, torch.from_numpy(s).cuda(), **opts).cpu().numpy()
    err = sampled_error(a, wl.grid, s, img, 31, 96 if wl is W.C3 else 256)
    print("   rel L2", err, flush=True)
    assert err < (1e-4 if precision == "fp32" else 1e-3)


def test_full_size_batch_of_pixel_per_lane_scans():
    wls = W.batch_c5()
    geoms = [pr.make_geometry(w.array) for w in wls]
    assert all(pr.hybrid_call_info(g, w.grid, **VECTOR).bp_kernel == "pixel-lanes" for g, w in zip(geoms, wls))
    batch = pr.HybridBatch(geoms, [w.grid for w in wls], VECTOR)
    assert batch.queued_scans == len(wls)
    echoes = [W.random_echo(w.array, 70 + i) for i, w in enumerate(wls)]
    print("batch: items", batch.work_items, flush=True)
    outs = pr.reconstruct_hybrid_batch(batch, [torch.from_numpy(e).cuda() for e in echoes])
    for i in (0, 7, 15):
        err = sampled_error(wls[i].array, wls[i].grid, echoes[i], outs[i].cpu().numpy(), 80 + i, 64)
        print("   scan", i, "rel L2", err, flush=True)
        assert err < 1e-4
