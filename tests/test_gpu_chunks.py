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
