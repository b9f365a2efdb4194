"""Modularity against the CPU oracle where rows, wave steps and wave ranges
begin and end: empty rows, rows longer than a range, one community, as many as
vertices, and labels that share slots of the workgroup's table.  All sums are
in fp64: relative to the sums' size 1e-12 a thousandfold covers their order."""
import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402


def star_and_ragged(n, spokes, hi, seed):
    """Symmetric graph: vertex n // 2 tied to the first `spokes` others, rows of
    0 .. about 2 hi entries besides, the last tenth of the vertices empty."""
    rng = np.random.default_rng(seed)
    live = max(n - n // 10, 1)
    src = np.repeat(np.arange(live), rng.integers(0, hi + 1, live))
    dst = rng.integers(0, live, len(src))
    src = np.concatenate([src, np.full(min(spokes, live), n // 2)])
    dst = np.concatenate([dst, np.arange(min(spokes, live))])
    keep = src != dst
    key = np.unique(np.concatenate([src[keep] * n + dst[keep], dst[keep] * n + src[keep]]))
    off = np.zeros(n + 1, dtype=np.int64)
    off[1:] = np.bincount(key // n, minlength=n)
    return np.cumsum(off), (key // n), (key % n).astype(np.int32)


@pytest.mark.parametrize("weights", ["unit", "int", "float"])
@pytest.mark.parametrize("n,spokes,hi", [(2, 1, 1), (70, 3, 2), (130, 127, 0), (258, 257, 0),
                                         (900, 300, 3), (5000, 10, 40), (300001, 250000, 1),
                                         (1500001, 1400000, 2)])
def test_sums(n, spokes, hi, weights):
    off, src, tgt = star_and_ragged(n, spokes, hi, n)
    w = np.ones(len(tgt), dtype=np.float32)
    if weights != "unit":
        a, b = np.minimum(src, tgt).astype(np.int64), np.maximum(src, tgt).astype(np.int64)
        w = (1 + (a * 31 + b * 17) % 8).astype(np.float32)
        if weights == "float":
            w = (w * np.float32(0.37) + np.float32(1e-3)).astype(np.float32)
    g = graphgen.Graph(off if weights == "int" else off.astype(np.int32), tgt, w)
    G = lpa.LpaGraph(*[torch.from_numpy(x).cuda() for x in (g.offsets, g.targets, g.weights)])
    rng = np.random.default_rng(7)
    ids = np.arange(n, dtype=np.uint64)
    slot = ids[((ids * 0x9E3779B1) % (1 << 32)) >> 22 == 5]  # one slot of the table
    for lab in (np.zeros(n), np.arange(n), rng.integers(0, n, n), np.arange(n) // 37,
                rng.choice(slot, n) if len(slot) else np.full(n, n - 1)):
        lab = lab.astype(np.int32)
        want = oracle.modularity(g.offsets, g.targets, g.weights, lab)
        got = G.modularity(torch.from_numpy(lab).cuda())
        assert got == pytest.approx(want, rel=1e-9, abs=1e-9)
    for bad in (-1, -7, n):
        lab = np.zeros(n, dtype=np.int32)
        lab[n // 2] = bad
        with pytest.raises(lpa.LpaError):
            G.modularity(torch.from_numpy(lab).cuda())
    G.close()
