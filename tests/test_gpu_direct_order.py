"""Direct evaluations of one context on several streams share its workspace: a
call that was refused has left the clearing of new counters on its stream,
which the next call on another stream must come after."""
import pytest

import oracle
import synth
from synth import Roi

pytestmark = pytest.mark.gpu

from gpu_common import check_density, dev, sfk, torch  # noqa: F401


def test_refused_call_comes_before_the_next_on_another_stream(sfk, torch, monkeypatch):
    pts = synth.clumpy_cloud(5_000, 3)
    roi = Roi((0.2,) * 3, (0.8,) * 3, (20,) * 3, bw="fixed", h=(0.05,) * 3)
    want = oracle.density(pts, roi)
    alloc = torch.cuda.caching_allocator_alloc
    calls, fail_at = [0], [-1]

    def take(n, device):
        calls[0] += 1
        return None if calls[0] == fail_at[0] else alloc(n, device)

    monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", take)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    out = torch.empty(roi.n_nodes, device="cuda")
    for k in range(1, 40):
        with sfk.Context(0) as c:
            tree = c.build_tree(dev(torch, pts))
            torch.cuda.synchronize()
            with torch.cuda.stream(s1):
                torch.cuda._sleep(30_000_000)
            fail_at[0] = calls[0] + k
            refused = False
            try:
                c.eval_roi(tree, roi, out=out, stream=s1)
            except sfk.SfkError as e:
                refused = e.status == 2  # SFK_E_NOMEM
                assert refused
            fail_at[0] = -1
            c.eval_roi(tree, roi, out=out, stream=s2)
            s2.synchronize()
            assert s1.query(), k
            check_density(out.cpu().numpy(), want, k)
            torch.cuda.synchronize()
            tree.close()
        if not refused:
            break
    assert k > 12 and not refused
