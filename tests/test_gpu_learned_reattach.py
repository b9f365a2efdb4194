"""State that outlives a learned run: a captured iteration after the same
predictor is attached with other options, the history after a refused run."""
import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402
from test_gpu_learned import (P_HISTORY, SMALL_TUNING, _assert_same, _gpu_graph,  # noqa: E402
                              _max_pred_degree, _min_pred_degree, _tuning)


def _oracle(g, tuning, small, large):
    return oracle.lpa_learned(g.offsets, g.targets, g.weights, params=P_HISTORY, z_theta=0.0,
                              pl_period=4, guard=4, fn_bound=1.0,
                              max_pred_degree=_max_pred_degree(tuning, large),
                              min_pred_degree=_min_pred_degree(tuning, small), pred_start=2)


@pytest.mark.parametrize("order", [[(0, 0), (1, 1)], [(1, 1), (0, 0)],
                                   [(0, 0), (1, 0), (0, 1), (0, 0)]])
@pytest.mark.parametrize("launch", [lpa.LAUNCH_GRAPH, lpa.LAUNCH_EAGER])
def test_classes_predicted_follow_the_attached_options(order, launch):
    g = graphgen.random_graph(3000, 0.033, seed=5, wmax=8)
    G = _gpu_graph(g, _tuning(**SMALL_TUNING))
    pr = lpa.Predictor(params=P_HISTORY)
    for small, large in order:
        G.set_predictor(pr, threshold=0.5, fn_bound=1.0, guard_period=4,
                        predict_small=bool(small), predict_large=bool(large))
        res = G.run("det", learned=True, launch=launch)
        _assert_same(_oracle(g, SMALL_TUNING, small, large), G, res)
    G.close()
    pr.close()


def test_history_survives_a_refused_run():
    g = graphgen.planted_partition_10k(1)
    G = _gpu_graph(g)
    pr = lpa.Predictor(params=P_HISTORY)
    G.set_predictor(pr, threshold=0.5, fn_bound=1.0)
    G.run("det", learned=True)
    kept = G.learned_history()
    assert len(kept) > 2 and kept[1]["iteration"] == 1
    bad = np.full(len(g.offsets) - 1, -1, dtype=np.int32)
    with pytest.raises(lpa.LpaError):
        G.run("det", learned=True, initial_labels=bad)
    assert G.learned_history() == kept
    G.run("det")                       # a plain run has none
    assert G.learned_history() == []
    G.close()
    pr.close()
