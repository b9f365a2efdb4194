"""Batched runs on the work queue at the edges of its kernel: row lengths where
a list or a 16-entry slice ends, chunks and graphs that share flag words, and
a graph with more vertices than the flag bits kept in LDS."""
import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402
from test_gpu_short_rows import circulant, graph  # noqa: E402


def check(graphs, chunk, group, launch, **kw):
    g, v_off = graphgen.pack_graphs(graphs)
    t = lpa.default_tuning()
    t.batch_queue, t.queue_chunk, t.queue_group = 1, chunk, group
    dev = [torch.from_numpy(x).cuda() for x in (g.offsets, g.targets, g.weights)]
    B = lpa.LpaBatch(v_off, *dev, tuning=t)
    res = B.run_batched("det", launch=launch, **kw)
    labels, flags = res.labels.cpu().numpy(), B.flags()
    for q, x in enumerate(graphs):
        ref = oracle.lpa_sync(x.offsets, x.targets, x.weights, **kw)
        part = slice(v_off[q], v_off[q + 1])
        assert res.iters_per_graph[q] == ref.iterations, q
        assert res.changed_last[q] == ref.stats[-1]["changed"], q
        assert np.array_equal(labels[part] - v_off[q], ref.labels), q
        # a vertex is flagged when a neighbour changed in the last iteration
        before = oracle.lpa_sync(x.offsets, x.targets, x.weights,
                                 **{**kw, "max_iterations": ref.iterations - 1}).labels \
            if ref.iterations > 1 else np.arange(len(ref.labels))
        moved = before != ref.labels
        src = np.repeat(np.arange(len(moved)), np.diff(x.offsets))
        want = np.zeros(len(moved), dtype=bool)
        np.logical_or.at(want, src, moved[x.targets])
        assert np.array_equal(flags[part].astype(bool), want), q
    B.close()


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("chunk,group,launch", [(64, 16, lpa.LAUNCH_EAGER),
                                                (512, 64, lpa.LAUNCH_GRAPH),
                                                (1024, 40, lpa.LAUNCH_EAGER)])
def test_row_lengths(chunk, group, launch, weighted):
    # vertex counts that are no multiple of 32, so that graphs and chunks
    # begin inside flag words
    graphs = [graph([circulant(n, d)], weighted)
              for d, n in [(1, 34), (2, 33), (15, 98), (16, 131), (17, 130), (31, 258), (32, 77),
                           (33, 260), (40, 95), (41, 98), (63, 66), (64, 67), (65, 1026),
                           (130, 263), (511, 514), (512, 1031)]]
    check(graphs, chunk, group, launch, max_iterations=5)


def test_more_vertices_than_flag_bits_in_lds():
    rng = np.random.default_rng(2)
    big = graph([circulant(70001, 6)], False)
    perm = rng.permutation(70001)                      # neighbours far apart
    src = np.repeat(np.arange(70001), 6)
    a, b = perm[src], perm[big.targets]
    order = np.lexsort((b, a))
    big = graphgen.Graph(big.offsets, b[order].astype(np.int32), big.weights)
    check([big, graph([circulant(97, 18)], False)], 512, 64, lpa.LAUNCH_GRAPH, max_iterations=6)
