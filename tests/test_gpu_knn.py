"""k-NN bandwidth at the edges of its candidate queue and merge networks: list
lengths either side of every register-array size, clouds of one to a few
leaves with a ragged last one, duplicates (ties and zero distances), and
cluster edges, where few lanes take most candidates. Bit-exact against the
oracle: the canonical float32 distances, selected without approximation."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

from gpu_common import ctx, dev, sfk, torch  # noqa: F401


def _cloud(kind, n, seed):
    g = np.random.default_rng(seed)
    if kind == "uniform":
        p = g.random((n, 3))
    elif kind == "clusters":  # tight clusters in a thin background
        c = g.random((5, 3))
        p = np.where(g.random(n)[:, None] < 0.1, g.random((n, 3)),
                     c[g.integers(0, 5, n)] + 1e-3 * g.standard_normal((n, 3)))
    else:  # a coarse lattice: many coincident points and tied distances
        p = g.integers(0, 6, (n, 3)) / 8.0
    return p.astype(np.float32)


@pytest.mark.parametrize("kind", ["uniform", "clusters", "lattice"])
@pytest.mark.parametrize("n", [66, 129, 1000, 20011])
def test_knn_bit_exact_at_edges(ctx, torch, kind, n):
    pts = _cloud(kind, n, n)
    for k in (1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 48, 63, 64):
        if k >= n:
            continue
        tree = ctx.build_tree(dev(torch, pts), knn_k=k)
        assert np.array_equal(ctx.debug_point_h2(tree), oracle.knn_h2(pts, k)), (kind, n, k)
        tree.close()
