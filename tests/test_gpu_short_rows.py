"""Rows of up to 64 entries: the 16-lane kernels against the CPU oracle at the
row lengths where a lane or a 16-entry slice begins or ends, with labels that
share slots of the match table, and at list lengths on both sides of each
batch size of the wave."""
import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402


def circulant(n, d, base=0):
    """Rows of d entries on n vertices: neighbours at distances 1 .. d/2, and
    the opposite vertex when d is odd (n even, d < n)."""
    v = np.arange(n)
    dist = [s for k in range(1, d // 2 + 1) for s in (k, n - k)] + ([n // 2] if d % 2 else [])
    tgt = np.sort((v[:, None] + np.array(dist, dtype=np.int64)) % n, axis=1) + base
    return tgt.astype(np.int32)


def graph(rows, weighted, offset_dtype=np.int32):
    """CSR of equal-length row blocks; integer weights 1 .. 8, equal both ways."""
    off = np.concatenate([[0], np.cumsum(np.concatenate([np.full(len(r), r.shape[1])
                                                         for r in rows]))])
    tgt = np.concatenate([r.ravel() for r in rows])
    src = np.repeat(np.arange(len(off) - 1), np.diff(off))
    w = np.ones(len(tgt), dtype=np.float32)
    if weighted:
        a, b = np.minimum(src, tgt).astype(np.int64), np.maximum(src, tgt).astype(np.int64)
        w = (1 + (a * 31 + b * 17) % 8).astype(np.float32)
    return graphgen.Graph(off.astype(offset_dtype), tgt, w)


def check(g, tuning=None, initial=None, **kw):
    ref = oracle.lpa_sync(g.offsets, g.targets, g.weights, initial_labels=initial, **kw)
    dev = [torch.from_numpy(x).cuda() for x in (g.offsets, g.targets, g.weights)]
    G = lpa.LpaGraph(*dev, tuning=tuning)
    res = G.run("det", initial_labels=None if initial is None
                else torch.from_numpy(initial).cuda(), **kw)
    assert res.iterations == ref.iterations
    for s_gpu, s_ref in zip(res.stats, ref.stats):
        for key in ("changed", "processed", "edges_scanned"):
            assert s_gpu[key] == s_ref[key], (key, s_gpu, s_ref)
    assert np.array_equal(res.labels.cpu().numpy(), ref.labels)
    G.close()


def tuning(**kw):
    t = lpa.default_tuning()
    for k, v in kw.items():
        setattr(t, k, v)
    return t


@pytest.mark.parametrize("labels", ["ids", "random", "one slot"])
@pytest.mark.parametrize("weighted,offset_dtype", [(False, np.int32), (True, np.int64)])
@pytest.mark.parametrize("small16", [16, 0])
def test_every_row_length(small16, weighted, offset_dtype, labels):
    # 98 rows of each length 1 .. 66; small16 = 0 sends the shortest rows
    # through the 17-64-entry kernel too
    rows = [circulant(98, d, 98 * (d - 1)) for d in range(1, 67)]
    g = graph(rows, weighted, offset_dtype)
    n = g.num_vertices
    init = None
    if labels == "random":
        init = np.random.default_rng(3).integers(0, n, n).astype(np.int32)
    elif labels == "one slot":  # labels that one hash slot holds in the first round
        ids = np.arange(n, dtype=np.uint64)
        same = ids[((ids * 0x9E3779B1) % (1 << 32)) >> 25 == 5]
        init = np.random.default_rng(4).choice(same, n).astype(np.int32)
    t = tuning(small4=min(4, small16), small16=small16)
    check(g, t, init, max_iterations=6)


def test_rows_with_self_loops():
    # a row whose own vertex is among its entries, at its start, middle and end
    n, rows = 200, []
    tgt = circulant(n, 20)
    off, out = [0], []
    for v in range(n):
        r = list(tgt[v]) + ([v] if v % 3 == 0 else [])
        out += sorted(r)
        off.append(len(out))
    g = graphgen.Graph(np.array(off, dtype=np.int32), np.array(out, dtype=np.int32),
                       np.ones(len(out), dtype=np.float32))
    check(g, initial=np.random.default_rng(5).integers(0, n, n).astype(np.int32))


# waves take 1, 2, 4, 8 or 16 rows a lane group and batch, by the list's length
@pytest.mark.parametrize("d", [6, 18])
@pytest.mark.parametrize("n", [33, 32768, 70003, 140001, 550001, 1600001])
def test_batch_sizes(n, d):
    check(graph([circulant(n, d)], weighted=n % 2 == 0), max_iterations=3)
