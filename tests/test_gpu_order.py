"""The tree's order at the edges of the sort: tiles of 4096 keys and their
remainders, one to eight passes of both key widths, ties (input order), and
more tiles than one round of a digit's row scan. Exact."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

from gpu_common import ctx, dev, sfk, torch  # noqa: F401
from test_gpu_parity import quantise_like_device


def _check(ctx, sfk, torch, pts, bits):
    tree = ctx.build_tree(dev(torch, pts), key_bits=bits)
    _, bbox, _ = tree.info()
    keys = sfk.curve_keys("hilbert", bits, quantise_like_device(pts, bbox, bits))
    order = ctx.debug_tree_order(tree)
    tree.close()
    assert np.array_equal(order, np.argsort(keys, kind="stable"))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1025, 4095, 4096, 4097, 12_289])
def test_order_at_tile_edges(ctx, sfk, torch, n):
    pts = synth.clumpy_cloud(max(n, 64), n)[:n]
    for bits in (1, 2, 5, 8, 10, 11, 16):
        _check(ctx, sfk, torch, pts, bits)


def test_order_with_many_tiles(ctx, sfk, torch):
    # 4097 tiles: a digit's row takes two rounds
    g = np.random.default_rng(3)
    pts = g.random((4096 * 4096 + 5, 3), dtype=np.float32)
    _check(ctx, sfk, torch, pts, 3)
