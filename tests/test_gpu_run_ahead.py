"""Iterations launched ahead of the stop: the same iterations, statistics and
labels as the CPU oracle at every cap and stop, eager and captured, also past
the statistics that a handle has room for from the start, and from handles of
several threads at once."""
import threading

import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402

KEYS = ("changed", "processed", "edges_scanned", "pick_less")


def bipartite(n):
    """Two sides that swap labels for ever: vertex v and its neighbours v + 1,
    v + 3, v - 1, v - 3 around an even ring."""
    v = np.arange(n)
    tgt = np.sort((v[:, None] + np.array([1, 3, n - 1, n - 3])) % n, axis=1).astype(np.int32)
    return graphgen.Graph(np.arange(0, 4 * n + 1, 4, dtype=np.int32), tgt.ravel(),
                          np.ones(4 * n, dtype=np.float32))


def handle(g):
    return lpa.LpaGraph(*[torch.from_numpy(x).cuda() for x in (g.offsets, g.targets, g.weights)])


def check(g, G, launch, **kw):
    ref = oracle.lpa_sync(g.offsets, g.targets, g.weights, **kw)
    res = G.run("det", launch=launch, **kw)
    assert res.iterations == ref.iterations
    assert len(res.stats) == len(ref.stats)
    for i, (s_gpu, s_ref) in enumerate(zip(res.stats, ref.stats)):
        assert s_gpu["iteration"] == i
        for key in KEYS:
            assert s_gpu[key] == s_ref[key], (i, key, s_gpu, s_ref)
        if launch == lpa.LAUNCH_EAGER:
            assert s_gpu["ms"] > 0
    assert np.array_equal(res.labels.cpu().numpy(), ref.labels)


@pytest.mark.parametrize("launch", [lpa.LAUNCH_EAGER, lpa.LAUNCH_GRAPH])
def test_caps(launch):
    g = bipartite(64)
    init = np.arange(64, dtype=np.int32) % 2
    G = handle(g)
    for cap in (0, 1, 2, 3, 5, 64, 65, 100, 7, 200):
        ref = oracle.lpa_sync(g.offsets, g.targets, g.weights, initial_labels=init,
                              max_iterations=cap, tolerance=0.0, pl_period=0)
        res = G.run("det", launch=launch, initial_labels=torch.from_numpy(init).cuda(),
                    max_iterations=cap, tolerance=0.0, pl_period=0)
        assert res.iterations == ref.iterations == cap
        assert [s["changed"] for s in res.stats] == [64] * cap
        assert [s["iteration"] for s in res.stats] == list(range(cap))
        assert np.array_equal(res.labels.cpu().numpy(), ref.labels)
    G.close()


@pytest.mark.parametrize("launch", [lpa.LAUNCH_EAGER, lpa.LAUNCH_GRAPH])
def test_stops(launch):
    g = graphgen.planted_partition_10k(3)
    G = handle(g)
    for tol in (0.9, 0.3, 0.05, 0.01, 0.0):
        for cap in (1, 4, 20):
            check(g, G, launch, tolerance=tol, max_iterations=cap)
    G.close()


def test_threads():
    graphs = [graphgen.planted_partition_10k(5), bipartite(2000), graphgen.rmat_graph(12, 6, "int8")]
    bad = []

    def work(g, launch):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                G = handle(g)
                torch.cuda.current_stream().synchronize()
                for cap in (3, 20, 12):
                    check(g, G, launch, max_iterations=cap, tolerance=0.01)
                G.close()
        except BaseException as e:  # shown by the main thread
            bad.append(e)

    ts = [threading.Thread(target=work, args=(g, la)) for g in graphs
          for la in (lpa.LAUNCH_EAGER, lpa.LAUNCH_GRAPH)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad
