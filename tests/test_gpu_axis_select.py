"""The in-box particle set and Eq. 1's order statistics at their edges: boxes
that cross zero (the widest key range: three digits), thin ones (one digit),
few particles, ties, and leaves that the box holds whole, cuts or misses. The
particle set and the lengths are exact (the same order statistics in the same
double arithmetic), so they are compared bit for bit with the oracle."""
import numpy as np
import pytest

import oracle
import synth
from synth import Roi

pytestmark = pytest.mark.gpu

from gpu_common import check_density, ctx, dev, sfk, torch  # noqa: F401


def _cloud(kind, n):
    rng = np.random.default_rng(n)
    if kind == "uniform":
        return rng.random((n, 3), dtype=np.float32), (0.1, 0.1, 0.1), (0.9, 0.9, 0.9)
    if kind == "signed":  # keys on both sides of zero, many octaves, both zeros
        p = (rng.random((n, 3)) * 2 - 1).astype(np.float32) ** 5
        p[: n // 8] = 0.0
        p[: n // 16] = -0.0
        return p, (-0.5, -1e-3, -0.7), (0.5, 0.9, 1e-4)
    if kind == "corner0":  # a corner at zero and negative zeros on it
        p = rng.random((n, 3)).astype(np.float32)
        p[: n // 4, 0] = -0.0
        return p, (0.0, 0.0, 0.25), (1.0, 0.5, 1.0)
    if kind == "thin":  # a handful of floats wide
        p = (np.float32(1.0) + rng.integers(0, 9, (n, 3)) * np.float32(2.0 ** -23)).astype(np.float32)
        return p, (1.0, 1.0, 1.0), (1.0 + 6 * 2.0 ** -23,) * 3
    p = np.full((n, 3), 0.25, np.float32)  # ties: P80 == P20 takes the cap
    p[: max(1, n // 10)] = rng.random((max(1, n // 10), 3), dtype=np.float32)
    return p, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0)


@pytest.mark.parametrize("n", [1, 2, 65, 1000, 70_003])
@pytest.mark.parametrize("kind", ["uniform", "signed", "corner0", "thin", "ties"])
def test_in_box_set_and_lengths(ctx, torch, kind, n):
    pts, lo, hi = _cloud(kind, n)
    roi = Roi(lo, hi, (6, 5, 7), bw="mbe", set="in_roi")
    tree = ctx.build_tree(dev(torch, pts))
    d = ctx.debug_mbe(tree, roi, cap_b=n)
    idx = np.nonzero(oracle.in_box_mask(pts, roi.lo, roi.hi))[0]
    assert d["n_b"] == len(idx)
    if len(idx):
        assert np.array_equal(np.asarray(d["idx_b"])[: len(idx)], idx)
        want, _ = oracle.mbe_initial_ell(pts[idx], roi)
        assert np.array_equal(d["ell0"], want)
    tree.close()


@pytest.mark.parametrize("lo,hi", [((0.0,) * 3, (1.0,) * 3), ((0.2, 0.3, 0.1), (0.8, 0.7, 0.9))])
def test_leaves_with_particles_without_support(ctx, torch, lo, hi):
    # particles whose k nearest coincide with them have no support and leave
    # their leaf's box: a leaf that the box holds whole then counts fewer
    pts = synth.clumpy_cloud(4_000, 5)
    pts[::3] = pts[0]
    tree = ctx.build_tree(dev(torch, pts), knn_k=8)
    h2 = ctx.debug_point_h2(tree)
    assert (h2 == 0).sum() > 1000
    roi = Roi(lo, hi, (9, 9, 9), bw="per_point", set="in_roi", norm="count")
    check_density(ctx.eval_roi(tree, roi).cpu().numpy(), oracle.density(pts, roi, h2=h2), "support")
    tree.close()
