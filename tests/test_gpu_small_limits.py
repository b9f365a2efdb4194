"""Small graphs under a memory limit of a few KiB: what a handle holds for the
graph counts, not the run state of a fixed size."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402


def _ring(n):
    v = np.arange(n)
    tgt = np.sort(np.stack([(v - 1) % n, (v + 1) % n], 1), 1).astype(np.int32).ravel()
    return torch.arange(0, 2 * n + 1, 2, dtype=torch.int32).cuda(), torch.from_numpy(tgt).cuda()


# bytes kept for a ring of n vertices on device arrays: at most 9 arrays of 4 n and
# 3 of n bytes, 16 n for modularity, and 1 KiB of counts; in the internal order
# another CSR, its targets' ids and two orders, 4 (n + 1 + 2 n + 2 n + 2 n) bytes; as
# a work queue labels and flags again and 4 KiB of queue counters
@pytest.mark.parametrize("n,relabel,batch,kib", [(3, 0, False, 3), (3, 1, False, 3), (3, 0, True, 7),
                                                 (64, 0, False, 6), (64, 1, False, 8),
                                                 (64, 0, True, 10), (500, 0, False, 24),
                                                 (500, 1, False, 38), (500, 0, True, 29),
                                                 (3000, 0, False, 130)])
def test_small_graphs_fit_small_limits(n, relabel, batch, kib):
    off, tgt = _ring(n)
    t = lpa.default_tuning()
    t.relabel = relabel
    free = lpa.LpaGraph(off, tgt, tuning=t)
    want = free.run("det").labels.cpu()
    t.memory_limit_kib = kib
    G = (lpa.LpaBatch(np.array([0, n]), off, tgt, tuning=t) if batch
         else lpa.LpaGraph(off, tgt, tuning=t))
    for launch in (lpa.LAUNCH_EAGER, lpa.LAUNCH_GRAPH):
        r = G.run("det", launch=launch)
        assert torch.equal(r.labels.cpu(), want)
    assert G.modularity(r.labels) == free.modularity(r.labels)
    G.close()
    free.close()
    t.memory_limit_kib = 1
    if n > 64:
        with pytest.raises(lpa.LpaError):
            lpa.LpaGraph(off, tgt, tuning=t)
