"""Wavefront tiles at their edges: the float32 cull must keep every particle
that reaches a node (exact support counts, at coordinates far from the origin
and for boxes of a single node), chunks of 32 and 256 leaves must give a ROI
the same grid alone and beside one of the other size, and tiles that walk the
hierarchy, per chunk or whole, must give the stored lists' grids bit for bit."""
import numpy as np
import pytest

import oracle
import synth
from synth import Roi

pytestmark = pytest.mark.gpu

from gpu_common import check_density, ctx, dev, sfk, torch  # noqa: F401


def _far_cloud(n, offset, seed):
    # particles on and within a few float steps of node distances, so many
    # pairs lie at the support's very edge
    g = np.random.default_rng(seed)
    p = g.random((n, 3)) + offset
    q = n // 2
    p[:q] = offset + g.integers(0, 17, (q, 3)) / 16.0
    f = p.astype(np.float32)
    f[: n // 4] = np.nextafter(f[: n // 4], np.float32(offset + 8.0))
    return f


@pytest.mark.parametrize("shape", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("offset", [0.0, 1000.0, -70000.0])
def test_cull_keeps_every_member(ctx, torch, shape, offset):
    pts = _far_cloud(3000, offset, 3)
    tree = ctx.build_tree(dev(torch, pts), knn_k=5)
    h2 = ctx.debug_point_h2(tree)
    lo, hi = (offset,) * 3, (offset + 1.0,) * 3
    ctx.set_eval_opts(tile_shape=shape)
    for kw in [dict(bw="fixed", h=(0.125, 0.0625, 0.25)),
               dict(bw="fixed", h=(0.01, 0.02, 0.003)),
               dict(bw="fixed", h=(0.0625,) * 3, kernel="gauss_trunc3"),
               dict(bw="per_point"), dict(bw="per_point", kernel="gauss_trunc3")]:
        roi = Roi(lo, hi, (9, 17, 6), norm="count", **kw)
        per = dict(h2=h2) if roi.bw == "per_point" else {}
        cnt = ctx.debug_support_counts(tree, roi).cpu().numpy().astype(np.int64)
        assert np.array_equal(cnt, oracle.support_counts(pts, roi, **per)), kw
        check_density(ctx.eval_roi(tree, roi).cpu().numpy(), oracle.density(pts, roi, **per), kw)
    ctx.set_eval_opts()
    tree.close()


@pytest.mark.parametrize("bw,kernel", [("per_point", "epanechnikov"), ("per_point", "gauss_trunc3"),
                                       ("fixed", "epanechnikov")])
def test_chunk_classes_alone_and_mixed(ctx, torch, bw, kernel):
    pts = synth.clumpy_cloud(120_000, 6)
    tree = ctx.build_tree(dev(torch, pts), knn_k=16)
    h = (0.03,) * 3 if bw == "fixed" else (0.0,) * 3
    # 25^3 = 15625 tiles of 4^3 and 26^3 = 17576: either side of 16384
    rois = [Roi((0.1,) * 3, (0.9,) * 3, (r,) * 3, bw=bw, kernel=kernel, h=h) for r in (100, 101, 30)]
    ctx.set_eval_opts(tile_shape=1)
    alone = [ctx.eval_roi(tree, r).cpu().numpy() for r in rois]
    outs = [torch.full((r.n_nodes,), -1.0, device="cuda") for r in rois]
    ctx.wait(ctx.submit(tree, rois, outs))
    for a, o, r in zip(alone, outs, rois):
        assert np.array_equal(a, o.cpu().numpy()), r.res
    # no list (every tile walks), with and without partial slots
    for kw in [dict(list_capacity=1), dict(list_capacity=1, partial_capacity=1 << 18),
               dict(list_capacity=20_000, partial_capacity=300)]:
        ctx.set_eval_opts(tile_shape=1, **kw)
        for a, r in zip(alone, rois):
            assert np.array_equal(a, ctx.eval_roi(tree, r).cpu().numpy()), (kw, r.res)
    ctx.set_eval_opts()
    tree.close()


@pytest.mark.parametrize("n", [1000, 2047 * 64, 2048 * 64])
def test_brick_chunk_classes_bitwise(ctx, torch, n):
    # few bricks over a small cloud take short chunks; 4 x 4 x 4 and 3 x 4 x 4
    # bricks lie either side of the line, as do the two larger clouds
    tree = ctx.build_tree(dev(torch, synth.clumpy_cloud(n, 8)))
    for res in [(16, 16, 16), (48, 64, 50), (64, 64, 49), (64, 64, 64)]:
        roi = Roi((0.05,) * 3, (0.95,) * 3, res, bw="fixed", h=(0.02,) * 3)
        ctx.set_eval_opts(tile_shape=6)
        a = ctx.eval_roi(tree, roi).cpu().numpy()
        out = torch.empty(roi.n_nodes, device="cuda")
        ctx.wait(ctx.submit(tree, [roi], [out]))
        ctx.set_eval_opts(tile_shape=6, chunk_leaves=256)
        b = ctx.eval_roi(tree, roi).cpu().numpy()
        assert np.array_equal(a, b) and np.array_equal(a, out.cpu().numpy()), res
    ctx.set_eval_opts()
    tree.close()


@pytest.mark.parametrize("h", [(0.4, 0.9, 0.3), (1.2, 1.2, 1.2), (1.4, 3.4, 0.6), (2.4, 1.0, 3.4),
                               (2.499, 2.5, 2.501), (2.6, 2.6, 2.6), (3.4, 0.7, 3.4),
                               (5.5, 6.5, 2.2)])
def test_brick_spans(ctx, torch, h):
    # supports of 1 to 14 nodes an axis, either side of the 6 in x that a
    # brick keeps in registers, on ragged bricks; up to 8 the sweep takes them
    pts = synth.clumpy_cloud(5000, 9)
    tree = ctx.build_tree(dev(torch, pts))
    roi = Roi((0.1, 0.2, 0.15), (0.9, 0.8, 0.95), (35, 18, 33), bw="fixed",
              h=tuple(v * s for v, s in zip(h, (0.8 / 34, 0.6 / 17, 0.8 / 32))))
    ctx.set_eval_opts(tile_shape=6)
    a = ctx.eval_roi(tree, roi).cpu().numpy()
    check_density(a, oracle.density(pts, roi), h)
    if max(h) < 3.5:
        ctx.set_eval_opts(tile_shape=7)
        assert np.array_equal(a, ctx.eval_roi(tree, roi).cpu().numpy())
    ctx.set_eval_opts()
    tree.close()
