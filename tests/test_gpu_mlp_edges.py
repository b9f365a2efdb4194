"""The change predictor's kernels at the edges of their splits: sample counts
around a round of 32, a group of 64 losses and the most workgroups, features
that are not 16-byte aligned, and a training step against its parts."""
import numpy as np
import pytest

from oracle import mlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2411_11468_amd import lpa  # noqa: E402
from test_gpu_predictor import _params, _samples  # noqa: E402


@pytest.mark.parametrize("n", [2, 31, 32, 33, 65, 8191, 8193, 16384, 16387, 50021])
def test_gradient_is_the_mean_over_its_parts(n):
    # a sample's activations do not depend on how the samples are split, so the
    # gradient of n samples is the weighted mean of those of any parts, up to
    # fp32 sums: a sum of n terms of both signs is off by at most about
    # sqrt(n) 2^-24 of the terms' root mean square, here below 1e-5 of the
    # largest gradient.  (Parts of up to 1,000 samples are held against the
    # fp64 oracle in test_gpu_predictor.py.  For many samples the oracle and
    # any fp32 forward pass may fall on different sides of a ReLU's kink.)
    p = _params(3)
    X, y = (torch.from_numpy(a).cuda() for a in _samples(n, n))
    pr = lpa.Predictor(params=mlp.flatten(p))
    g, loss = pr.gradient(X, y, pos_weight=1.5)
    cuts = sorted({0, n // 3, 2 * n // 3, n})
    mean, mean_loss = np.zeros(mlp.N_PARAMS), 0.0
    for a, b in zip(cuts[:-1], cuts[1:]):
        gp, lp = pr.gradient(X[a:b].contiguous(), y[a:b].contiguous(), pos_weight=1.5)
        mean += gp.astype(np.float64) * (b - a) / n
        mean_loss += lp * (b - a) / n
    assert loss == pytest.approx(mean_loss, rel=1e-6)
    np.testing.assert_allclose(g, mean, rtol=0, atol=1e-5 * np.abs(mean).max())
    pr.close()


@pytest.mark.parametrize("n,batch", [(700, 700), (4099, 5000)])
def test_one_training_step_is_gradient_and_adam(n, batch):
    # the same samples in another order: the gradients agree to fp32 rounding,
    # and a first Adam step moves each parameter by lr g / (|g| + eps), so a
    # relative error of 1e-4 in g moves it by less than lr 1e-4
    p = mlp.flatten(_params(5))
    X, y = (torch.from_numpy(a).cuda() for a in _samples(n, 9))
    a, b = lpa.Predictor(params=p), lpa.Predictor(params=p)
    loss_a = a.train(X, y, epochs=1, batch=batch, lr=1e-3, pos_weight=2.0, seed=1)
    g, loss_b = b.gradient(X, y, pos_weight=2.0)
    b.adam(lr=1e-3)
    assert loss_a == pytest.approx(loss_b, rel=1e-5)
    big = np.abs(g) > 1e-4 * np.abs(g).max()   # gradients above their rounding error
    np.testing.assert_allclose(a.params()[big], b.params()[big], rtol=2e-7, atol=2e-6)
    a.close()
    b.close()


@pytest.mark.parametrize("n", [1, 17, 64 * 1024, 64 * 1024 + 1, 300007])
def test_predict_unaligned_features(n):
    p = lpa.Predictor(params=mlp.flatten(_params(2)))
    X, _ = _samples(n, 4)
    flat = torch.zeros(12 * n + 1, device="cuda")
    flat[1:] = torch.from_numpy(X).cuda().ravel()
    shifted = flat[1:].view(n, 12)
    assert shifted.data_ptr() % 16 == 4
    got = p.predict(shifted)
    assert torch.equal(got, p.predict(torch.from_numpy(X).cuda()))
    z, _ = mlp.forward(mlp.unflatten(p.params()), X, bf16_h1=True)
    # as in test_gpu_predictor.py: rare flips of a bf16 rounding aside
    err = np.abs(got.cpu().numpy() - mlp.sigmoid(z))
    assert np.mean(err > 1e-4) <= max(0.05, 1.0 / n)
    p.close()
