"""Ordered selections at the edges of their words and tiles, capacities below
the count, and sampling where the box's magnitudes allow the reciprocal
division and where they don't. Exact: both sides round the same operations."""
import ctypes as C

import numpy as np
import pytest

import oracle
import synth
from synth import Roi

pytestmark = pytest.mark.gpu

from gpu_common import ctx, dev, sfk, torch  # noqa: F401


@pytest.mark.parametrize("n", [1, 63, 64, 65, 2047, 2048, 2049, 6145])
def test_select_tile_edges_and_capacities(ctx, torch, sfk, n):
    import paper_2601_20758_amd._lib as L
    roi = Roi((0.1, -0.3, 0.25), (0.9, 0.55, 1.4), (9, 8, 7))
    grid = synth.random_grid(roi.res, 4)
    pts = synth.probe_points(roi, 7000, 5)[:n]
    g_d, p_d = dev(torch, grid), dev(torch, pts)
    for iso in (-1.0, 1.0):
        ref = oracle.select_points(grid, roi, iso, pts)
        for cap in sorted({0, 1, len(ref) // 2, max(0, len(ref) - 1), len(ref), n}):
            idx = torch.full((n + 1,), -7, dtype=torch.int64, device="cuda")
            cnt = C.c_int64()
            r = sfk.roi_struct(roi, 0)
            assert L.lib().sfk_select_points(ctx._h, C.byref(r), g_d.data_ptr(), iso,
                                             p_d.data_ptr(), n, idx.data_ptr(), cap, C.byref(cnt),
                                             None) == 0
            got = idx.cpu().numpy()
            m = min(cap, len(ref))
            assert cnt.value == len(ref) and np.array_equal(got[:m], ref[:m])
            assert (got[m:] == -7).all()


@pytest.mark.parametrize("res", [(2, 2, 2), (2, 3, 1025), (65, 2, 33), (3, 65, 17), (14, 13, 15)])
def test_iso_tile_edges_and_capacities(ctx, torch, sfk, res):
    import paper_2601_20758_amd._lib as L
    roi = Roi((0.0, -1.0, 2.0), (1.0, 1.0, 2.5), res)
    grid = synth.random_grid(res, 6)
    g_d = dev(torch, grid)
    for iso in (float(np.quantile(grid, 0.02)), float(np.median(grid)), float(grid.max()) + 1.0):
        rc, rk = oracle.iso_cells(grid, roi, iso)
        tri = np.asarray(oracle.iso_surface(grid, roi, iso), np.float32).reshape(-1, 9)
        for part in (0, 1, 2):
            r = sfk.roi_struct(roi, 0)
            cnt = C.c_int64()
            cap = len(rc) * part // 2
            cells = torch.full((len(rc) + 1,), -7, dtype=torch.int64, device="cuda")
            cases = torch.full((len(rc) + 1,), 77, dtype=torch.uint8, device="cuda")
            assert L.lib().sfk_iso_cells(ctx._h, C.byref(r), g_d.data_ptr(), iso,
                                         cells.data_ptr(), cases.data_ptr(), cap, C.byref(cnt),
                                         None) == 0
            assert cnt.value == len(rc)
            assert np.array_equal(cells.cpu().numpy()[:cap], rc[:cap])
            assert np.array_equal(cases.cpu().numpy()[:cap], rk[:cap])
            assert (cells[cap:] == -7).all() and (cases[cap:] == 77).all()
            cap = len(tri) * part // 2
            out = torch.full((len(tri) + 1, 9), -7.0, device="cuda")
            assert L.lib().sfk_iso_surface(ctx._h, C.byref(r), g_d.data_ptr(), iso, out.data_ptr(),
                                           cap, C.byref(cnt), None) == 0
            assert cnt.value == len(tri) and np.array_equal(out.cpu().numpy()[:cap], tri[:cap])
            assert (out[cap:] == -7).all()


@pytest.mark.parametrize("lo,hi", [
    ((0.0, 0.1, -0.7), (1.0 / 3.0, 0.3, 0.9)),
    ((1e-30, -1e-30, 0.0), (3e-30, 1e-30, 7e-31)),
    ((1e6, -3e7, 65536.0), (1e6 + 1.0, -2.9e7, 65537.0)),
    ((-1e300, 0.0, 0.0), (1e300, 1.0, 1.0)),      # span 2e300: plain division
    ((1e-150, 0.0, 0.0), (1.0, 1.0, 1.0)),        # corner below the range: plain division
    ((-1e38, -1e38, -3e38), (1e38, 2e38, 3e38)),
])
def test_sampling_at_all_magnitudes(ctx, torch, lo, hi):
    roi = Roi(lo, hi, (33, 100, 77))
    grid = synth.random_grid(roi.res, 8)
    g = np.random.default_rng(9)
    lo64, hi64 = np.array(lo), np.array(hi)
    p = lo64 + g.random((20_000, 3)) * (hi64 - lo64)
    k = g.integers(0, 3, 4000)  # on lattice planes and corners too
    node = lo64 + np.round(g.random((4000, 3)) * 32) * ((hi64 - lo64) / 32)
    p[:4000][np.arange(4000), k] = node[np.arange(4000), k]
    with np.errstate(over="ignore"):
        pts = p.astype(np.float32)
    pts = pts[np.isfinite(pts).all(axis=1)]
    if len(pts) == 0:
        pts = np.zeros((100, 3), np.float32) + g.random((100, 3)).astype(np.float32)
    got = ctx.sample_density(roi, dev(torch, grid), dev(torch, pts)).cpu().numpy()
    assert np.array_equal(got, oracle.sample_density(grid, roi, pts).astype(np.float32))
