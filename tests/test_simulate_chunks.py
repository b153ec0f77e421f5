"""Echo simulation: frequency chunks, scatterer runs and both arrays.

Tolerance 4e-6 relative L2 against float64: phasors of three hardware sines
(absolute error up to 2^-20) and at most five float32 products, sums of 32 in
float32.  Edges: chunks of 16 and 32 frequencies with full and ragged last
ones, runs of 32 scatterers, thread counts on both sides of the rule.
"""
import os
from dataclasses import replace

import pytest

import workloads as W
from oracle import geometry as ogeom

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pr = pytest.importorskip("paper_2109_02842_amd")

TOL = 4e-6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pr.LIB_PATH):
        pytest.fail("libpolyrecon.so is not built")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("mode", ["mono", "multi"])
@pytest.mark.parametrize("n_freq,n_scat,n_scan", [(1, 1, 5), (15, 31, 9), (16, 32, 8), (17, 33, 8), (33, 2, 7),
                                                  (51, 65, 9), (64, 3, 1400), (100, 3, 1000), (40, 3, 1400)])
def test_simulated_echo_against_float64(mode, n_freq, n_scat, n_scan):
    a = replace(W.C1.array, n_freq=n_freq, n_scan=n_scan, scan_step=0.001)
    if mode == "multi":
        a = replace(a, mode="multi", spacing=W._D_MULTI, n_tx=2)
    geom = pr.make_geometry(a)
    arr = ogeom.build(a)
    gen = torch.Generator().manual_seed(7)
    xyz = ((torch.rand(n_scat, 3, generator=gen, dtype=torch.float64) - 0.5) * 0.3).cuda()
    refl = torch.complex(torch.randn(n_scat, generator=gen, dtype=torch.float64),
                         torch.randn(n_scat, generator=gen, dtype=torch.float64)).cuda()
    print(mode, n_freq, n_scat, n_scan, flush=True)
    got = pr.simulate_echo(geom, xyz, refl)
    d = lambda v: torch.from_numpy(v).cuda()
    z, k = d(arr.z_scan), d(arr.k)
    ref = torch.zeros(geom.echo_shape, dtype=torch.complex128, device="cuda")
    for s in range(n_scat):
        dz2 = (xyz[s, 2] - z)[None] ** 2
        path = sum((((xyz[s, :2] - d(p)) ** 2).sum(1)[:, None] + dz2).sqrt() for p in (arr.tx, arr.rx))
        ref += refl[s] * torch.exp(-1j * path[:, :, None] * k)
    err = float((got - ref).norm() / ref.norm())
    print("   rel L2", err, flush=True)
    assert err < TOL
    assert float(pr.simulate_echo(geom, xyz[:0], refl[:0]).abs().max()) == 0.0
