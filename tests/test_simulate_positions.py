"""Echo simulation at positions off the ordinary range.

A coordinate that is not a number or infinite gives an echo that is not a
number in every sample (each sample sums every scatterer).  A position whose
squared distance passes the float32 range has a finite echo of its
reflectivity's size.  Paths of 1e6 m keep float64 accuracy: the phase of 1.4e9
rad carries a few float64 roundings (2^-52 each, 1e-6 rad in all) beside the
4e-6 that the float32 phasors and sums are held to elsewhere.
"""
import math
import os
from dataclasses import replace

import pytest

import workloads as W
from oracle import geometry as ogeom

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


def array(mode):
    a = replace(W.C1.array, n_chords=1, n_elem=4, n_freq=19, n_scan=6)
    return replace(a, mode="multi", spacing=W._D_MULTI, n_tx=2) if mode == "multi" else a


def simulate(a, xyz, refl):
    return pr.simulate_echo(pr.make_geometry(a), torch.tensor(xyz, dtype=torch.float64, device="cuda"),
                            torch.tensor(refl, dtype=torch.complex128, device="cuda"))


@pytest.mark.parametrize("mode", ["mono", "multi"])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("value", [math.nan, math.inf])
def test_a_position_that_is_no_number_reaches_every_sample(mode, axis, value):
    xyz = [[0.1, 0.0, 0.0], [0.0, 0.1, 0.02]]
    xyz[1][axis] = value
    print(mode, axis, value, flush=True)
    assert bool(torch.isnan(simulate(array(mode), xyz, [1.0, 1.0])).all())


@pytest.mark.parametrize("mode", ["mono", "multi"])
def test_a_far_position_keeps_a_finite_echo(mode):
    got = simulate(array(mode), [[1e20, 0.0, 0.0]], [2.0 - 1.0j])
    print(mode, float((got.abs() - 5 ** 0.5).abs().max()), flush=True)
    assert bool(torch.isfinite(torch.view_as_real(got)).all())
    assert float((got.abs() - 5 ** 0.5).abs().max()) < 1e-5


@pytest.mark.parametrize("mode", ["mono", "multi"])
def test_paths_of_1e6_m_keep_float64_accuracy(mode):
    a = array(mode)
    arr = ogeom.build(a)
    gen = torch.Generator().manual_seed(3)
    xyz = (torch.rand(40, 3, generator=gen, dtype=torch.float64) - 0.5) * 1e6
    got = simulate(a, xyz.tolist(), [1.0] * 40).cpu().to(torch.complex128)
    ref = torch.zeros_like(got)
    z, k = torch.from_numpy(arr.z_scan), torch.from_numpy(arr.k)
    for p in xyz:
        dz2 = (p[2] - z)[None] ** 2
        path = sum((((p[:2] - torch.from_numpy(q)) ** 2).sum(1)[:, None] + dz2).sqrt() for q in (arr.tx, arr.rx))
        ref += torch.exp(-1j * path[:, :, None] * k)
    err = float((got - ref).norm() / ref.norm())
    print(mode, "rel L2", err, flush=True)
    assert err < 5e-6
