"""The order of the gradient's sums.  Training rounds the weights to bf16 at
every step, so one ulp of a gradient can move later steps by 2^-9 of a weight:
the gradient is held to the bit against chains of fused multiply-adds over each
64 samples in their order, the parts added in fp64, and an epoch of training to
the bit against one gradient and one Adam step per minibatch.

A fused multiply-add of floats is emulated in 80-bit arithmetic: the product is
exact there, and the sum is rounded at 64 bits before it is rounded to 24
(differently from one rounding about once in 2^40)."""
import ctypes
import subprocess

import numpy as np
import pytest

from oracle import mlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402
from test_gpu_predictor import _params, _samples  # noqa: E402

f32, wide = np.float32, np.longdouble


def _fma(a, b, c):
    return (a.astype(wide) * b.astype(wide) + c.astype(wide)).astype(f32)


def _chain(a, b, start):
    """start + a[0] * b[0] + a[1] * b[1] + ..., one fused multiply-add each."""
    acc = np.broadcast_to(start, np.broadcast_shapes(a.shape[1:], b.shape[1:])).astype(f32)
    for x, y in zip(a, b):
        acc = _fma(x, y, acc)
    return acc


def _gradient_of_64(p, X, dz):
    """Gradient of at most 64 samples, d loss / d logit given."""
    W1, W2, W3, x = (mlp.bf16_round(a) for a in (p["W1"], p["W2"], p["W3"], X))
    h1 = np.maximum(_chain(x.T[:, :, None], W1[:, None, :], p["b1"]), f32(0))
    h2 = np.maximum(_chain(h1.T[:, :, None], W2[:, None, :], p["b2"]), f32(0))
    da2 = np.where(h2 > 0, dz[:, None] * W3[:, 0][None, :], f32(0)).astype(f32)
    da1 = _chain(da2.T[:, :, None], W2.T[:, None, :], f32(0))
    da1 = np.where(h1 > 0, da1, f32(0))
    one = np.ones(len(dz), dtype=f32)
    g = {"W1": _chain(x[:, :, None], da1[:, None, :], f32(0)), "b1": _chain(da1, one, f32(0)),
         "W2": _chain(h1[:, :, None], da2[:, None, :], f32(0)), "b2": _chain(da2, one, f32(0)),
         "W3": _chain(h2, dz, f32(0)), "b3": _chain(dz, one, f32(0))}
    return mlp.flatten(g)


@pytest.mark.parametrize("n", [1, 33, 64, 65, 200])
def test_gradient_sums_in_sample_order(n):
    p = _params(3)
    X, y = _samples(n, 40 + n)
    pr = lpa.Predictor(params=mlp.flatten(p))
    g, _ = pr.gradient(X, y, pos_weight=1.5)
    # a sample's d loss / d logit is its gradient of b3 alone, up to the factor 1 / n
    one = [pr.gradient(X[s:s + 1], y[s:s + 1], pos_weight=1.5)[0][-1] for s in range(n)]
    dz = np.array(one, dtype=f32) * (f32(1) / f32(n))
    total = np.zeros(mlp.N_PARAMS)
    for s in range(0, n, 64):
        total += _gradient_of_64(p, X[s:s + 64], dz[s:s + 64]).astype(np.float64)
    np.testing.assert_array_equal(g, total.astype(f32))
    pr.close()


@pytest.mark.parametrize("parts", [2, 64, 512])
def test_gradient_adds_its_parts_in_64_bits(parts):
    # for a power of two the factor 1 / n scales every sum without rounding
    p = _params(6)
    n = 64 * parts
    X, y = (torch.from_numpy(a).cuda() for a in _samples(n, parts))
    pr = lpa.Predictor(params=mlp.flatten(p))
    g, _ = pr.gradient(X, y, pos_weight=2.0)
    total = np.zeros(mlp.N_PARAMS)
    for s in range(0, n, 64):
        gp, _ = pr.gradient(X[s:s + 64], y[s:s + 64], pos_weight=2.0)
        total += gp.astype(np.float64) / parts
    np.testing.assert_array_equal(g, total.astype(f32))
    pr.close()


@pytest.fixture(scope="module")
def shuffles(tmp_path_factory):
    """Sample orders of the epochs: std::shuffle on std::mt19937_64(seed)."""
    d = tmp_path_factory.mktemp("shuffle")
    (d / "s.cpp").write_text("""
#include <algorithm>
#include <cstdint>
#include <numeric>
#include <random>
#include <vector>
extern "C" void shuffles(uint64_t seed, int64_t n, int32_t epochs, int32_t* out) {
  std::vector<int32_t> perm(n);
  std::iota(perm.begin(), perm.end(), 0);
  std::mt19937_64 rng(seed);
  for (int32_t e = 0; e < epochs; ++e) {
    std::shuffle(perm.begin(), perm.end(), rng);
    std::copy(perm.begin(), perm.end(), out + e * n);
  }
}
""")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", str(d / "s.cpp"), "-o",
                           str(d / "s.so")])
    lib = ctypes.CDLL(str(d / "s.so"))

    def call(seed, n, epochs):
        out = np.empty((epochs, n), dtype=np.int32)
        lib.shuffles(ctypes.c_uint64(seed), ctypes.c_int64(n), ctypes.c_int32(epochs),
                     out.ctypes.data_as(ctypes.c_void_p))
        return out
    return call


@pytest.mark.parametrize("n,batch,epochs", [(1000, 256, 2), (1001, 100, 1), (70001, 33000, 1)])
def test_training_is_gradient_and_adam_per_minibatch(shuffles, n, batch, epochs):
    start = mlp.flatten(_params(5))
    X, y = (torch.from_numpy(a).cuda() for a in _samples(n, 9))
    trained = []
    for _ in range(2):
        a = lpa.Predictor(params=start)
        loss = a.train(X, y, epochs=epochs, batch=batch, lr=1e-3, pos_weight=2.0, seed=11)
        trained.append((a.params(), loss, a.save_blob()))
        a.close()
    b = lpa.Predictor(params=start)
    for order in shuffles(11, n, epochs):
        total = 0.0
        for s in range(0, n, batch):
            i = torch.from_numpy(order[s:s + batch].astype(np.int64)).cuda()
            _, mean = b.gradient(X[i], y[i], pos_weight=2.0)
            b.adam(lr=1e-3)
            total += mean * len(i)
    for params, loss, blob in trained:
        np.testing.assert_array_equal(params, b.params())
        assert blob == b.save_blob()
        assert loss == pytest.approx(total / n, rel=1e-6)   # a float
    assert trained[0][1] == trained[1][1]
    b.close()
