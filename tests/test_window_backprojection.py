"""The whole-call FP32 back-projection on the matrix cores (window form).

Tolerance 3e-5 relative L2 against the float64 oracle: the planner takes this
form only where its interpolation error is below 0.55 (even window starts) or
0.9 (any start) of the B-spline's, whose estimate is at most 2.3e-5 at six
times oversampling (sqrt(2) (1/12)^4 / 3); the roundings (FP16 pairs, 2^-22 of
each product; NUFFT tolerance 1e-6) add below 5e-6.
"""
import math
import os
from dataclasses import replace

import numpy as np
import pytest

import workloads as W
from oracle import geometry as ogeom
from oracle import hybrid as ohyb

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pr = pytest.importorskip("paper_2109_02842_amd")

TOL = 3e-5


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pr.LIB_PATH):
        pytest.fail("libpolyrecon.so is not built")
    yield
    torch.cuda.synchronize()


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def grid(nx, ny, d):
    return W.ImageGrid(nx=nx, ny=ny, x0=-d * (nx - 1) / 2 + 0.004, y0=-d * (ny - 1) / 2 - 0.003, dx=d, dy=d)


MONO = replace(W.C1.array, n_scan=229, n_elem=17, n_freq=20)          # 51 channels: a lone last one
MULTI = W.ArrayDesc(mode="multi", n_chords=3, radius=0.5, n_elem=11, spacing=W._D_MULTI, n_tx=2, n_scan=230,
                    scan_step=0.005, n_freq=16, f_start=26e9, f_stop=34e9)   # 66 channels

# (array, grid): partial tiles and pixel groups, odd scan lengths (rows without
# a mirror), one and several k_z blocks, fine pixels (even window starts) and
# coarser ones (any start), monostatic and multistatic
CASES = {
    "mono-fine": (MONO, grid(45, 29, 0.0026)),
    "mono-coarse": (MONO, grid(45, 29, 0.0046)),
    "mono-one-tile": (MONO, grid(13, 15, 0.003)),
    "mono-331": (replace(MONO, n_scan=331), grid(30, 48, 0.003)),
    "multi-fine": (MULTI, grid(27, 47, 0.0024)),
    "multi-coarse": (MULTI, grid(15, 62, 0.0038)),
}


def window_and_steps(name, s):
    a, g = CASES[name]
    geom = pr.make_geometry(a)
    whole = pr.reconstruct_hybrid(geom, g, dev(s))
    valu = pr.reconstruct_hybrid(geom, g, dev(s), mfma_backprojection=-1)   # an asked-for kernel: the other path
    assert not torch.equal(whole, valu), "the whole call did not take the window form"
    return host(whole), host(valu)


@pytest.mark.parametrize("name", sorted(CASES))
def test_window_against_oracle_and_the_other_path(name):
    a, g = CASES[name]
    s = W.random_echo(a, 5)
    whole, valu = window_and_steps(name, s)
    ref = ohyb.image(ogeom.build(a), g, s)
    e, ev = rel(whole, ref), rel(valu, ref)
    print(name, "rel L2", e, "other path", ev, flush=True)
    assert e < TOL


@pytest.mark.parametrize("scale", [1e-15, 1.0, 1e15])
def test_window_follows_the_data_scale(scale):
    # the profiles' power of two comes from the spectrum
    a, g = CASES["mono-fine"]
    s = W.random_echo(a, 6)
    geom = pr.make_geometry(a)
    ref = ohyb.image(ogeom.build(a), g, s)
    got = host(pr.reconstruct_hybrid(geom, g, dev((s * scale).astype(np.complex64)))).astype(np.complex128) / scale
    assert rel(got, ref) < TOL
    zero = pr.reconstruct_hybrid(geom, g, dev(np.zeros_like(s)))
    assert float(zero.abs().max()) == 0.0
    s[3, 4, 5] = math.nan
    bad = pr.reconstruct_hybrid(geom, g, dev(s))
    assert not bool(torch.isfinite(bad).any())     # a NaN of one channel reaches every voxel


def test_window_batch_is_the_single_calls():
    names = sorted(CASES)
    geoms = [pr.make_geometry(CASES[n][0]) for n in names]
    echoes = [dev(W.random_echo(CASES[n][0], 70 + i)) for i, n in enumerate(names)]
    # one scan with an asked-for kernel: both queues in one call
    opts = [{} if n != "mono-one-tile" else dict(mfma_backprojection=-1) for n in names]
    batch = pr.HybridBatch(geoms, [CASES[n][1] for n in names], opts)
    for i, out in enumerate(pr.reconstruct_hybrid_batch(batch, echoes)):
        single = pr.reconstruct_hybrid(geoms[i], CASES[names[i]][1], echoes[i], **opts[i])
        assert torch.equal(out, single), names[i]


@pytest.mark.parametrize("precision,mbp", [("bf16", 1), ("fp16", 1), ("bf16", 0), ("fp16", 0)])
@pytest.mark.parametrize("nx,ny,window", [(64, 64, True), (63, 65, False), (181, 131, True)])
def test_split_modes_take_the_window_form(precision, mbp, nx, ny, window):
    # from 4096 pixels on the modes run their FP32 plan's window form
    a, g = replace(MONO, n_elem=5, n_scan=224), grid(nx, ny, 0.0024)
    geom = pr.make_geometry(a)
    echo = dev(W.random_echo(a, 4))
    got = pr.reconstruct_hybrid(geom, g, echo, precision=precision, mfma_backprojection=mbp)
    assert torch.equal(got, pr.reconstruct_hybrid(geom, g, echo)) == window
    if not mbp:   # an asked-for kernel keeps the mode's own plan
        own = pr.reconstruct_hybrid(geom, g, echo, precision=precision, mfma_backprojection=-1)
        assert torch.equal(got, own) != window and rel(host(got), host(own)) < TOL
