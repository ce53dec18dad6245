"""Work items of wavefront tiles and bricks: regions of both chunk classes are
one group of one batch, and however few partial slots or list entries there
are, the grids are the same bit for bit."""
import numpy as np
import pytest

import synth
from synth import Roi

pytestmark = pytest.mark.gpu

from gpu_common import ctx, dev, sfk, torch  # noqa: F401


def test_chunk_classes_are_one_group(ctx, torch):
    # 4096 and 17576 tiles of 4^3, either side of the classes' line
    pts = synth.clumpy_cloud(50_000, 6)
    tree = ctx.build_tree(dev(torch, pts), knn_k=8)
    rois = [Roi((0.1,) * 3, (0.9,) * 3, (r,) * 3, bw="per_point") for r in (64, 104, 32, 101)]
    alone = [ctx.eval_roi(tree, r).cpu().numpy() for r in rois]
    outs = [torch.empty(r.n_nodes, device="cuda") for r in rois]
    ctx.profile_enable(True)
    ctx.profile_read(reset=True)
    ctx.wait(ctx.submit(tree, rois, outs))
    assert ctx.profile_read()["eval_launches"] == 1
    ctx.profile_enable(False)
    # and through one captured graph, in turn
    for _ in range(3):
        for a, o, r in zip(alone, outs, rois):
            o.fill_(-1.0)
            ctx.wait(ctx.submit(tree, [r], [o]))
            assert np.array_equal(a, o.cpu().numpy())
    tree.close()


def _grids(ctx, tree, rois, shape, **opts):
    ctx.set_eval_opts(tile_shape=shape, **opts)
    out = [ctx.eval_roi(tree, r).cpu().numpy() for r in rois]
    ctx.set_eval_opts()
    return out


# 1000 and 1728 tiles of 4^3, either side of the plan's 1024 in one launch
@pytest.mark.parametrize("shape,res", [(1, 40), (1, 48), (2, 33), (3, 30), (4, 20), (5, 11),
                                       (6, 40), (6, 170)])
def test_scarce_slots_and_lists_bitwise(ctx, torch, shape, res):
    pts = synth.clumpy_cloud(120_000, 7)
    tree = ctx.build_tree(dev(torch, pts), knn_k=8)
    # supports that reach most of a tile's neighbourhood: up to dozens of chunks
    h = (0.11, 0.2, 0.15) if shape < 6 else (0.03, 0.02, 0.025)
    rois = [Roi((0.05,) * 3, (0.95,) * 3, (res, res - 1, res), bw="fixed", h=h),
            Roi((0.3,) * 3, (0.7,) * 3, (res,) * 3, bw="fixed", h=h, kernel="gauss_trunc3")]
    if shape < 6:
        rois.append(Roi((0.2,) * 3, (0.8,) * 3, (res,) * 3, bw="per_point"))
    want = _grids(ctx, tree, rois, shape, partial_capacity=1 << (20 if shape < 6 else 11))
    lists = dict(list_capacity=1 << 22)
    for kw in [dict(partial_capacity=1, **lists), dict(partial_capacity=60, **lists),
               dict(partial_capacity=3000, **lists), dict(partial_capacity=1, list_capacity=1),
               dict(partial_capacity=60, list_capacity=3000),
               dict(partial_capacity=3000, list_capacity=40_000), dict(list_capacity=3000)]:
        for a, b, r in zip(want, _grids(ctx, tree, rois, shape, **kw), rois):
            assert np.array_equal(a, b), (kw, r)
    for a, r in zip(want, rois):
        ctx.set_eval_opts(tile_shape=shape)
        out = torch.full((r.n_nodes,), -1.0, device="cuda")
        ctx.eval_roi_noalloc(tree, r, out)
        assert np.array_equal(a, out.cpu().numpy())
        ctx.set_eval_opts()
    tree.close()


@pytest.mark.parametrize("shape", [1, 6])
def test_lists_are_exported_without_slots(ctx, torch, shape):
    tree = ctx.build_tree(dev(torch, synth.clumpy_cloud(120_000, 7)))
    roi = Roi((0.05,) * 3, (0.95,) * 3, (60,) * 3, bw="fixed", h=(0.05,) * 3)
    ctx.set_eval_opts(tile_shape=shape)
    _, cnt, leaves = ctx.debug_tile_leaves(tree, roi)
    assert cnt.max() > 64  # more than a chunk of either shape: some tiles are split
    ctx.set_eval_opts(tile_shape=shape, partial_capacity=1, list_capacity=1 << 22)
    _, cnt1, leaves1 = ctx.debug_tile_leaves(tree, roi)
    assert np.array_equal(cnt, cnt1) and np.array_equal(leaves, leaves1)
    ctx.set_eval_opts()
    tree.close()


@pytest.mark.parametrize("shape,res", [(6, 40), (6, 150), (1, 40)])
def test_list_capacity_bounds_the_slots(sfk, torch, shape, res):
    # 2^24 list entries: 65536 slots, 2 GiB of a brick's, whatever the chunks
    pts = synth.clumpy_cloud(20_000, 3)
    roi = Roi((0.1,) * 3, (0.9,) * 3, (res,) * 3, bw="fixed", h=(0.02,) * 3)
    grids = []
    for kw in [dict(budget_bytes=(2 << 30) + (256 << 20)), dict()]:
        with sfk.Context(0, **kw) as c:
            tree = c.build_tree(dev(torch, pts))
            c.set_eval_opts(tile_shape=shape, list_capacity=1 << 24 if kw else 0)
            grids.append(c.eval_roi(tree, roi).cpu().numpy())
            tree.close()
    assert np.array_equal(*grids)


def test_budgeted_batch_is_accepted_again(sfk, torch):
    # a chunk-heavy per-point batch in the budget its first call needs: what it
    # lacked must not make the next calls ask for more than there is
    pts = synth.clumpy_cloud(400_000, 5)
    rois = [Roi((0.05,) * 3, (0.95,) * 3, (48,) * 3, bw="per_point"),
            Roi((0.2,) * 3, (0.6,) * 3, (40,) * 3, bw="per_point"),
            Roi((0.05,) * 3, (0.95,) * 3, (48,) * 3, bw="fixed", h=(0.2,) * 3)]
    outs = [torch.empty(r.n_nodes, device="cuda") for r in rois]
    want, low = None, None
    for mb in (1 << 12, *range(16, 400, 4)):
        with sfk.Context(0, budget_bytes=mb << 20) as c:
            tree = c.build_tree(dev(torch, pts), knn_k=48)
            c.set_eval_opts(tile_shape=1)
            try:
                c.wait(c.submit(tree, rois, outs))
            except sfk.SfkError as e:
                assert e.status == 3  # SFK_E_BUDGET: below what a first call needs
                tree.close()
                continue
            got = [o.cpu().numpy() for o in outs]
            if want is None:
                want = got
            for _ in range(4):
                c.wait(c.submit(tree, rois, outs))
                for a, o in zip(want, outs):
                    assert np.array_equal(a, o.cpu().numpy()), mb
                    o.fill_(-1.0)
            tree.close()
            if mb < 1 << 12:
                low = low or mb
                if mb > low + 60:
                    break
    assert low is not None


def test_batch_memory_is_bounded(sfk, torch):
    # 3.5M tiles of short chunks: slots for a bounded number of them
    pts = synth.clumpy_cloud(50_000, 5)
    free = lambda: torch.cuda.mem_get_info()[0]
    used = []
    for count in (4, 256):
        rois = [Roi((0.1,) * 3, (0.3,) * 3, (96,) * 3, bw="per_point")] * count
        out = torch.empty((count, rois[0].n_nodes), device="cuda")
        torch.cuda.synchronize()
        with sfk.Context(0, allocator="hip") as c:
            tree = c.build_tree(dev(torch, pts), knn_k=8)
            c.set_eval_opts(disable_graphs=True)
            a = free()
            c.wait(c.submit(tree, rois, list(out)))
            used.append(a - free())
            assert bool((out == out[0]).all())
            tree.close()
        del out
    # per tile: lists of 64 leaves, a quarter of a slot of 512 B, counts and the
    # count pass's 256 leaves; 131072 slots for short chunks beside that
    tiles = 256 * 24 ** 3
    assert used[1] - used[0] < tiles * (64 * 4 + 512 // 4 + 256 * 4 + 64 + 512 // 2) + (64 << 20)
