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



class _Memory:
    """torch's allocator as a context sees it: it refuses call `fail_at` with
    work left on `stream`, and notes what is on it when memory comes back."""

    def __init__(self, torch, monkeypatch, stream):
        self.calls, self.fail_at, self.idle_at_free = 0, -1, []
        alloc, free = torch.cuda.caching_allocator_alloc, torch.cuda.caching_allocator_delete

        def take(n, device):
            self.calls += 1
            if self.calls == self.fail_at:
                with torch.cuda.stream(stream):
                    torch.cuda._sleep(30_000_000)
                return None
            return alloc(n, device)

        def give(p):
            if 0 <= self.fail_at <= self.calls:
                self.idle_at_free.append(stream.query())
            free(p)

        monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", take)
        monkeypatch.setattr(torch.cuda, "caching_allocator_delete", give)


@pytest.mark.parametrize("bw", ["mbe", "fixed", "per_point"])
def test_nothing_is_given_back_while_kernels_run(sfk, torch, monkeypatch, bw):
    # each allocation of an in-box evaluation refused once: the call fails only
    # when its stream is done with what it gives back
    pts = synth.clumpy_cloud(20_000, 3)
    roi = Roi((0.2,) * 3, (0.8,) * 3, (20,) * 3, bw=bw, set="in_roi", h=(0.05,) * 3)
    s = torch.cuda.Stream()
    mem = _Memory(torch, monkeypatch, s)
    out = torch.empty(roi.n_nodes, device="cuda")
    refused, last = 0, False
    for k in range(1, 80):
        with sfk.Context(0) as c:
            tree = c.build_tree(dev(torch, pts), knn_k=5 if bw == "per_point" else 0)
            torch.cuda.synchronize()
            mem.fail_at, mem.idle_at_free = mem.calls + k, []
            try:
                c.eval_roi(tree, roi, out=out, stream=s)
            except sfk.SfkError as e:
                assert e.status == 2 and s.query(), k  # SFK_E_NOMEM
            assert all(mem.idle_at_free), k
            last = mem.calls < mem.fail_at
            mem.fail_at = -1
            torch.cuda.synchronize()
            tree.close()
        if last:
            break
        refused += 1
    assert last and refused >= 10


@pytest.mark.parametrize("bw", ["mbe", "fixed", "per_point"])
def test_scratch_makes_room_for_the_grid(sfk, torch, monkeypatch, bw):
    # a few particles of a large cloud: the scratch over the cloud's leaves, the
    # evaluation's first three allocations, is given back when the grid's own
    # memory does not fit beside it
    pts = synth.clumpy_cloud(3_000_000, 4)
    roi = Roi((0.4,) * 3, (0.5,) * 3, (24,) * 3, bw=bw, set="in_roi", h=(0.01,) * 3)
    alloc, free = torch.cuda.caching_allocator_alloc, torch.cuda.caching_allocator_delete
    held, calls, need, limit = {}, [0], [0], [None]

    def take(n, device):
        calls[0] += 1
        used = sum(b for b, _ in held.values()) + n
        if limit[0] is not None and used > limit[0]:
            return None
        p = alloc(n, device)
        held[p] = n, calls[0]
        if calls[0] > 8:  # past the sub-cloud
            used -= sum(b for b, i in held.values() if 1 <= i <= 3)
        need[0] = max(need[0], used)
        return p

    def give(p):
        held.pop(p)
        free(p)

    monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", take)
    monkeypatch.setattr(torch.cuda, "caching_allocator_delete", give)
    grids, room = [], None
    for _ in range(2):
        with sfk.Context(0) as c:
            calls[0] = -10_000
            tree = c.build_tree(dev(torch, pts), knn_k=5 if bw == "per_point" else 0)
            limit[0], need[0], calls[0] = room, 0, 0
            grids.append(c.eval_roi(tree, roi).cpu().numpy())
            limit[0], room, calls[0] = None, need[0], -10_000
            tree.close()
    assert np.array_equal(*grids)
