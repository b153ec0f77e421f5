"""The window form's profile scale follows echoes down to the smallest floats.

Tolerance 3e-5 relative L2 against float64, as at ordinary scales: at 1e-39 the
echo keeps 19 significant bits (spacing 1.4e-45) and enters the reference as
rounded, the scan transform's values near 1e-38 round by 1e-44 in all (1e-6).
"""
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


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pr.LIB_PATH):
        pytest.fail("libpolyrecon.so is not built")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("scale", [1e-33, 1e-36, 1e-39])
def test_window_keeps_its_accuracy_at_the_smallest_scales(scale):
    a = replace(W.C1.array, n_scan=229, n_elem=17, n_freq=20)
    d = 0.0026
    grid = W.ImageGrid(nx=45, ny=29, x0=-d * 22 + 0.004, y0=-d * 14 - 0.003, dx=d, dy=d)
    s = (W.random_echo(a, 6) * scale).astype(np.complex64)
    geom, echo = pr.make_geometry(a), torch.from_numpy(s).cuda()
    ref = ohyb.image(ogeom.build(a), grid, s.astype(np.complex128) / scale)
    whole = pr.reconstruct_hybrid(geom, grid, echo)
    vector = pr.reconstruct_hybrid(geom, grid, echo, mfma_backprojection=-1)
    assert not torch.equal(whole, vector), "the whole call did not take the window form"
    err = [float(np.linalg.norm(t.cpu().numpy().astype(np.complex128) / scale - ref) / np.linalg.norm(ref))
           for t in (whole, vector)]
    print(scale, "rel L2", err[0], "vector kernels", err[1], flush=True)
    assert err[0] < 3e-5
