"""Rows of 65 entries and more, a wave each: matched in registers up to 256
entries and in a table beyond, against the CPU oracle at the lengths where a
64-entry slice, the registers or the class end, with labels that share slots."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_short_rows import check, circulant, graph, tuning  # noqa: E402

LENGTHS = (65, 66, 127, 128, 129, 191, 192, 193, 255, 256, 257, 319, 320, 511, 512, 513)


@pytest.mark.parametrize("labels", ["ids", "random", "few", "one slot"])
@pytest.mark.parametrize("weighted,offset_dtype", [(False, np.int32), (True, np.int64)])
@pytest.mark.parametrize("probe", [0, 1])
def test_lengths(probe, weighted, offset_dtype, labels):
    size = 530
    g = graph([circulant(size, d, size * i) for i, d in enumerate(LENGTHS)], weighted, offset_dtype)
    n = g.num_vertices
    rng = np.random.default_rng(3)
    init = None
    if labels == "random":
        init = rng.integers(0, n, n).astype(np.int32)
    elif labels == "few":
        init = rng.integers(0, 5, n).astype(np.int32)
    elif labels == "one slot":  # labels that one of the 512 slots holds in the first round
        ids = np.arange(n, dtype=np.uint64)
        same = ids[((ids * 0x9E3779B1) % (1 << 32)) >> 23 == 5]
        init = rng.choice(same, n).astype(np.int32)
    check(g, tuning(probe=probe), init, max_iterations=5)
