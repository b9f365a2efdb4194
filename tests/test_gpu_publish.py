"""Labels published and flags set after the sweeps, against the CPU oracle, at
vertex counts around the words, wave steps and grids of those kernels."""
import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402


def ragged(n, seed, hi):
    """Symmetric graph whose rows have 0 .. about 2 hi entries, one long row."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, hi + 1, n)
    src = np.repeat(np.arange(n), deg)
    dst = rng.integers(0, n, len(src))
    if n > 90:
        src = np.concatenate([src, np.zeros(80, dtype=src.dtype)])
        dst = np.concatenate([dst, np.arange(1, 81) * (n // 81)])
    keep = src != dst
    key = np.unique(np.concatenate([src[keep] * n + dst[keep], dst[keep] * n + src[keep]]))
    off = np.zeros(n + 1, dtype=np.int32)
    np.add.at(off, key // n + 1, 1)
    return graphgen.Graph(np.cumsum(off, dtype=np.int32), (key % n).astype(np.int32),
                          np.ones(len(key), dtype=np.float32))


@pytest.mark.parametrize("flag_mode", [lpa.FLAGS_PUSH, lpa.FLAGS_PULL])
@pytest.mark.parametrize("n,hi", [(1, 1), (2, 1), (31, 2), (33, 3), (63, 2), (65, 9), (511, 2),
                                  (513, 40), (2049, 3), (70001, 6), (1050001, 2)])
def test_labels_and_flags(n, hi, flag_mode):
    g = ragged(n, n, hi)
    dev = [torch.from_numpy(x).cuda() for x in (g.offsets, g.targets, g.weights)]
    G = lpa.LpaGraph(*dev)
    for iters in (1, 2, 3, 5):
        ref = oracle.lpa_sync(g.offsets, g.targets, g.weights, max_iterations=iters,
                              tolerance=0.0)
        res = G.run("det", max_iterations=iters, tolerance=0.0, flag_mode=flag_mode)
        assert np.array_equal(res.labels.cpu().numpy(), ref.labels)
        for s_gpu, s_ref in zip(res.stats, ref.stats):
            for key in ("changed", "processed", "edges_scanned"):
                assert s_gpu[key] == s_ref[key], (iters, key, s_gpu, s_ref)
    # the flags a next iteration would start from: the processed count of the
    # oracle's next iteration
    flags = G.flags().astype(bool)
    ref = oracle.lpa_sync(g.offsets, g.targets, g.weights, max_iterations=6, tolerance=0.0)
    if len(ref.stats) > 5:
        assert int(flags.sum()) == ref.stats[5]["processed"]
    G.close()
