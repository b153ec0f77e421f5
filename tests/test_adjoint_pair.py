"""Operator pairs of the differentiable calls on a plan whose whole calls take
the window form.

The echo model, its gradient and the refinement use one operator and its exact
transpose: <H y, x> = <y, H^H x> to 2e-6, the float32 roundings of both sides
(each side's relative error, near 1e-6, times |<.,.>| over the product of the
norms, which is below 1; the bound the other adjoint tests use).  Two operators
1e-5 apart pass that line too where their difference is nearly orthogonal to the
pair, so the operator itself is compared with the vector kernels' bit by bit.
The imaging call keeps the window form unless the caller asks for the vector
kernels: its gradient is then the transpose of an operator that differs from it
by both interpolation errors, 2.3e-5 and 1.05 of that at most.
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


ARRAY = replace(W.C1.array, n_scan=229, n_elem=9, n_freq=20)
GRID = W.ImageGrid(nx=45, ny=29, x0=-0.053, y0=-0.039, dx=0.0026, dy=0.0026)


@pytest.fixture(scope="module")
def geom():
    return pr.make_geometry(ARRAY)


def random(shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.view_as_complex(torch.randn(*shape, 2, device="cuda", generator=g))


def mismatch(a, b, c, d):
    """|<a, b> - <c, d>| over |a| |b| (float64)."""
    dot = lambda x, y: torch.vdot(x.reshape(-1).to(torch.complex128), y.reshape(-1).to(torch.complex128))
    norm = lambda x: float(x.reshape(-1).to(torch.complex128).norm())
    return abs(complex(dot(a, b) - dot(c, d))) / (norm(a) * norm(b))


def pulled_back(fn, x, y):
    """fn(x), and what backward gives x for the gradient y of fn(x)."""
    x = x.detach().clone().requires_grad_(True)
    out = fn(x)
    out.backward(y)
    return out.detach(), x.grad


def test_the_default_call_takes_the_window_form(geom):
    echo = random(geom.echo_shape, 1)
    assert not torch.equal(pr.reconstruct_hybrid(geom, GRID, echo),
                           pr.reconstruct_hybrid(geom, GRID, echo, mfma_backprojection=-1))


def test_echo_model_and_its_gradient_are_transposes(geom):
    from paper_2109_02842_amd import autograd as ag
    x, y = random((ARRAY.n_scan, GRID.ny, GRID.nx), 2), random(geom.echo_shape, 3)
    s, g = pulled_back(lambda v: ag.echo_model(geom, GRID, v), x, y)
    m = mismatch(y, s, g, x)
    # the part of <y, H^H x> that a random pair has: the adjoint error shows at full size for y = H^H x
    s2, g2 = pulled_back(lambda v: ag.echo_model(geom, GRID, v), x, s)
    m2 = mismatch(s2, s2, g2, x)
    print("echo model", m, m2, flush=True)
    assert m < 2e-6 and m2 < 2e-6
    assert torch.equal(g, pr.reconstruct_hybrid(geom, GRID, y, mfma_backprojection=-1))


def test_imaging_call_and_its_gradient(geom):
    from paper_2109_02842_amd import autograd as ag
    s, x = random(geom.echo_shape, 4), random((ARRAY.n_scan, GRID.ny, GRID.nx), 5)
    for opts, tol in ((dict(mfma_backprojection=-1), 2e-6), ({}, 2.3e-5 * 2.05)):
        img, _ = pulled_back(lambda v: ag.reconstruct(geom, GRID, v, **opts), s, x)
        img, g = pulled_back(lambda v: ag.reconstruct(geom, GRID, v, **opts), s, img)
        m = mismatch(img, img, g, s)
        print("imaging", opts, m, flush=True)
        assert m < tol
        assert torch.equal(img, pr.reconstruct_hybrid(geom, GRID, s, **opts))


@pytest.mark.parametrize("method", ["cg", "sd"])
def test_refinement_runs_the_exact_pair(geom, method):
    from paper_2109_02842_amd import autograd as ag
    s = pr.adjoint_hybrid(geom, GRID, random((ARRAY.n_scan, GRID.ny, GRID.nx), 6))
    a, ha = ag.refine(geom, GRID, s, steps=3, method=method)
    b, hb = ag.refine(geom, GRID, s, steps=3, method=method, mfma_backprojection=-1)
    assert torch.equal(a, b) and ha == hb
