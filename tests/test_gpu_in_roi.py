"""In-box sets with per-point bandwidths on ragged last leaves: the padding
slots of the sub-cloud must reach no node (exact support counts)."""
import numpy as np
import pytest

import oracle
import synth
from synth import Roi

pytestmark = pytest.mark.gpu

from gpu_common import check_density, ctx, dev, sfk, torch  # noqa: F401


@pytest.mark.parametrize("n", [64, 65, 100, 127, 3000])
@pytest.mark.parametrize("kernel", ["epanechnikov", "gauss_trunc3"])
def test_support_counts_on_a_ragged_last_leaf(ctx, torch, n, kernel):
    pts = synth.clumpy_cloud(n, n)
    tree = ctx.build_tree(dev(torch, pts), knn_k=5)
    h2 = ctx.debug_point_h2(tree)
    for lo, hi in [((0.0,) * 3, (1.0,) * 3), ((0.1, 0.2, 0.05), (0.8, 0.9, 0.95))]:
        roi = Roi(lo, hi, (9, 7, 11), bw="per_point", set="in_roi", kernel=kernel)
        cnt = ctx.debug_support_counts(tree, roi).cpu().numpy().astype(np.int64)
        assert np.array_equal(cnt, oracle.support_counts(pts, roi, h2=h2)), (lo, hi)
        check_density(ctx.eval_roi(tree, roi).cpu().numpy(), oracle.density(pts, roi, h2=h2), lo)
    tree.close()
