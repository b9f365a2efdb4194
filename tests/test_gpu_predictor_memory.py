"""A predictor holds device memory for gradients only once it computes them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402
from test_gpu_predictor import _samples  # noqa: E402


def test_predictors_that_never_train_hold_no_gradient_parts():
    X, _ = _samples(16, 1)
    lpa.Predictor(seed=0).predict(X)    # the library's own first allocations
    free = torch.cuda.mem_get_info()[0]
    many = [lpa.Predictor(seed=s) for s in range(64)]
    for p in many:
        p.predict(X)
    held = free - torch.cuda.mem_get_info()[0]
    # 0.1 MB of parameters, moments and operand tiles each, in blocks that the
    # allocator may round up to 2 MiB
    assert held <= 64 * 2 * 2 ** 20, held
    for p in many:
        p.close()


def test_gradient_space_grows_and_is_kept():
    X, y = _samples(40000, 2)
    a, b = lpa.Predictor(seed=1), lpa.Predictor(seed=1)
    want = [b.gradient(X[:n], y[:n])[0] for n in (40000, 64, 4096)]   # largest first
    got = [a.gradient(X[:n], y[:n])[0] for n in (64, 4096, 40000)]
    np.testing.assert_array_equal(got[0], want[1])
    np.testing.assert_array_equal(got[1], want[2])
    np.testing.assert_array_equal(got[2], want[0])
    a.close()
    b.close()
