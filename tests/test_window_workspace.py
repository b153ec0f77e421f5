"""Workspace of plans that take the window form (CPU only).

The spectrum and the image's spectrum are the vector plan's, the profiles are
on a coarser range grid; beside them the window form has its tables and, only
where the launch splits the work items past the last full round of 512, a
partial spectrum of 128 KiB per piece, at most 512 pieces.
"""
from dataclasses import replace

import pytest

import workloads as W

pr = pytest.importorskip("paper_2109_02842_amd")


def case(n_scan, nx, ny, n_elem=16, pitch=0.0028):
    a = replace(W.C1.array, n_scan=n_scan, n_elem=n_elem, n_freq=20, scan_step=0.004)
    return a, W.ImageGrid(nx=nx, ny=ny, x0=-pitch * (nx - 1) / 2, y0=-pitch * (ny - 1) / 2, dx=pitch, dy=pitch)


def sizes(a, grid):
    """Workspace of the whole call and of the vector plan, bytes of the window
    form's tables (tile table, 12 bytes per (k_z, frequency), rounding), items."""
    g = pr.make_geometry(a)
    tiles, blocks = -(-grid.nx // 16) * -(-grid.ny // 16), -(-((a.n_scan + 1) // 2) // 32)
    tables = tiles * g.n_channels * (48 + 8 * blocks) + 12 * a.n_scan * a.n_freq + (256 << 10)
    return (pr.hybrid_workspace_bytes(g, grid), pr.hybrid_workspace_bytes(g, grid, mfma_backprojection=-1), tables,
            tiles * blocks)


@pytest.mark.parametrize("n_scan,nx,ny", [(192, 208, 208), (250, 128, 256), (256, 256, 256), (130, 200, 160)])
def test_no_piece_is_held_where_no_item_is_split(n_scan, nx, ny):
    a, grid = case(n_scan, nx, ny)
    whole, vector, tables, items = sizes(a, grid)
    assert items % 512 == 0 or 2 * (items % 512) > 512
    assert whole <= vector + tables


@pytest.mark.parametrize("n_scan,nx,ny,n_elem", [(192, 96, 96, 16), (250, 208, 190, 5)])
def test_split_items_hold_their_pieces(n_scan, nx, ny, n_elem):
    a, grid = case(n_scan, nx, ny, n_elem)
    whole, vector, tables, items = sizes(a, grid)
    tail = items % 512
    pairs = (3 * n_elem + 1) // 2
    assert 0 < 2 * tail <= 512
    assert whole <= vector + tables + tail * min(512 // tail, pairs) * (128 << 10)


@pytest.mark.parametrize("n_scan,nx,ny,n_elem,n_freq", [(300, 150, 60, 40, 240), (200, 120, 90, 60, 256)])
def test_pieces_take_the_place_of_the_spectrum(n_scan, nx, ny, n_elem, n_freq):
    # a spectrum larger than all pieces: nothing is added for them
    a, grid = case(n_scan, nx, ny, n_elem)
    whole, vector, tables, items = sizes(replace(a, n_freq=n_freq), grid)
    assert 0 < 2 * (items % 512) <= 512 and 3 * n_elem * n_scan * n_freq * 8 >= 512 * (128 << 10)
    assert vector < whole <= vector + tables
