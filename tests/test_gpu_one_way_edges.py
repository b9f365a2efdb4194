"""Pulled flags where some targets have no entries of their own (edges stored in
one direction only): the internal order keeps such vertices behind those that
the change bits cover, so they must read as unchanged.  The caller's order,
which covers every vertex, gives the expected labels and counts."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402


def _one_way(n, sinks, seed):
    """Rows of 0-9 distinct sorted targets; the vertices in `sinks` have none."""
    rng = np.random.default_rng(seed)
    src = np.repeat(np.arange(n), 6)
    near = (src // 40 * 40 + rng.integers(0, 40, src.size)) % n
    dst = np.where(rng.random(src.size) < 0.5, near, rng.integers(0, n, src.size))
    keep = ~sinks[src] & (src != dst)
    key = np.unique(src[keep].astype(np.int64) * n + dst[keep])
    off = np.zeros(n + 1, dtype=np.int32)
    np.cumsum(np.bincount(key // n, minlength=n), out=off[1:])
    return off, (key % n).astype(np.int32)


# bits in LDS with 4 and with 16 waves a workgroup, and read from memory
@pytest.mark.parametrize("n", [3001, 300007, 1900003])
@pytest.mark.parametrize("profile", [False, True])
def test_targets_without_entries_read_as_unchanged(n, profile):
    rng = np.random.default_rng(n)
    off, tgt = _one_way(n, rng.random(n) < 0.3, n)
    runs = []
    for relabel in (0, 1):
        t = lpa.default_tuning()
        t.relabel = relabel
        G = lpa.LpaGraph(torch.from_numpy(off).cuda(), torch.from_numpy(tgt).cuda(), tuning=t)
        r = G.run("det", flag_mode=lpa.FLAGS_PULL, tolerance=0.0, profile=profile)
        runs.append((r.labels.cpu().numpy(), r.iterations,
                     [(s["changed"], s["processed"], s["edges_scanned"]) for s in r.stats],
                     G.flags()))
        G.close()
    (la, ia, sa, fa), (lb, ib, sb, fb) = runs
    assert ia == ib and sa == sb and ia > 4
    np.testing.assert_array_equal(la, lb)
    np.testing.assert_array_equal(np.asarray(torch.as_tensor(fa).cpu()),
                                  np.asarray(torch.as_tensor(fb).cpu()))
