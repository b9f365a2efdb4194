"""The profile's algorithmic bytes: what each kernel has to move, from counts
that the test knows itself."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402


def _ring(n, wide):
    off = np.arange(0, 2 * n + 1, 2).astype(np.int64 if wide else np.int32)
    v = np.arange(n)
    tgt = np.sort(np.stack([(v - 1) % n, (v + 1) % n], 1), 1).astype(np.int32)
    return torch.from_numpy(off).cuda(), torch.from_numpy(tgt.ravel()).cuda()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("mode", ["det", "async"])
def test_short_rows_flags_and_labels(mode, wide):
    # one class of kernels, labels given (so that they are gathered), the flags
    # pulled, one iteration that is not the last (the last pulls none)
    n = 5000
    G = lpa.LpaGraph(*_ring(n, wide))
    labels = torch.arange(n, dtype=torch.int32).cuda().flip(0).contiguous()
    G.profile_reset()
    r = G.run(mode, initial_labels=labels, max_iterations=2, tolerance=0.0, profile=True,
              flag_mode=lpa.FLAGS_PULL)
    prof = {p["name"]: p for p in G.profile()}
    changed = [s["changed"] for s in r.stats]
    verts = sum(s["processed"] for s in r.stats)
    assert r.iterations == 2 and changed[0] > 0
    ob = 16 if wide else 8
    # target and label per entry; list id, offsets and own label per vertex; new
    # label and change byte per change
    assert prof["sweep_small4"]["bytes"] == 8 * 2 * verts + (4 + ob + 4) * verts + 5 * sum(changed)
    # offset, class and flag per vertex, the change bits, the targets read
    scanned = prof["pull_flags"]["edges"]
    assert 0 < scanned <= 2 * n
    assert prof["pull_flags"]["bytes"] == n * (ob / 2 + 2) + n / 8 + 4 * scanned
    # change bytes read, bits written once; deterministic: the labels copied
    assert prof["apply"]["bytes"] == (2 * n + 8 * sum(changed) if mode == "det" else n) + n / 8
    G.close()


def test_work_queue_rows():
    v_off = np.arange(0, 4001, 1000)
    off, tgt = _ring(1000, False)
    k = len(v_off) - 1
    off = torch.cat([off[:1]] + [off[1:] + 2000 * q for q in range(k)]).contiguous()
    tgt = torch.cat([tgt + 1000 * q for q in range(k)]).contiguous()
    t = lpa.default_tuning()
    t.batch_queue = 1
    B = lpa.LpaBatch(v_off, off, tgt, tuning=t)
    labels = torch.cat([torch.arange(1000 * q, 1000 * q + 1000, dtype=torch.int32).flip(0)
                        for q in range(k)]).cuda()
    for mode in ("det", "async"):
        B.profile_reset()
        r = B.run(mode, initial_labels=labels, max_iterations=1, tolerance=0.0, profile=True)
        prof = {p["name"]: p for p in B.profile()}
        n = 4000
        # a flag bit per vertex; offsets and own label per processed vertex; new
        # label per change
        want = 8 * 2 * n + n / 8 + (8 + 4) * n + 4 * r.stats[0]["changed"]
        assert prof["queue_sweep"]["bytes"] == want
    B.close()
