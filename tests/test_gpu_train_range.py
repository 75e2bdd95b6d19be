"""Training gradients with saturated units: pre-activations so large that the GELU
and its derivative are exactly z and 1, or 0 and 0."""
import numpy as np
import pytest

import oracle
from test_gpu_train_net import TOL, dev, f32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("big", [20.0, 1e4, 1e12, 1e14, 1e18])
def test_gradient_with_saturated_units(big):
    """Even units of layer 1 at +big (columns of W2 over big, so layer 2 is of
    order one), odd ones at -big.  The even units' gradients to the bound of the
    other network tests; the odd ones', zero in FP64, to the sum of 64 products
    with the smallest factors that the kernels form: |z| 2^-126 in the GELU,
    60 |z| 2^-126 in its derivative."""
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] training network, pre-activations {big}", flush=True)
    n = 100
    rng = np.random.default_rng(7)
    w1 = rng.standard_normal((64, 8)) / np.sqrt(8)
    b1 = np.where(np.arange(64) % 2, -big, big)
    w2 = rng.standard_normal((64, 64)) / np.sqrt(64)
    w2[:, ::2] /= big
    p = np.concatenate([w1.ravel(), b1, w2.ravel(), 0.1 * rng.standard_normal(64),
                        rng.standard_normal(192) / np.sqrt(64), 0.1 * rng.standard_normal(3)])
    nm = np.concatenate([np.zeros(8), np.ones(8), [1e-4, 2e-4, 1e-4]])
    p, nm = f32(p), f32(nm)
    x = f32(rng.standard_normal((n, 8)))
    t = f32(1e-4 * rng.standard_normal((n, 3)))
    loss_ref, ref = oracle.mlp_loss_grad(p, nm, x, t / nm[16:19])
    tr = rrmhd.Trainer(n)
    grad = torch.empty(4931, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    tr.loss_grad(dev(p), dev(nm), dev(x), dev(t), grad, loss)
    got = grad.cpu().numpy().astype(np.float64)
    tr.close()
    assert abs(loss.item() - loss_ref) < TOL * abs(loss_ref)

    def parts(v):
        w1, b1, w2 = v[:512].reshape(64, 8), v[512:576], v[576:4672].reshape(64, 64)
        return ([w1[::2], b1[::2], w2[:, ::2], v[4672:4736], v[4736:4928], v[4928:]],
                [w1[1::2], b1[1::2], w2[:, 1::2]])

    for g, r in zip(parts(got)[0], parts(ref)[0]):
        assert np.linalg.norm(g - r) < TOL * np.linalg.norm(r)
    small = 64 * 60 * big * 2.0 ** -126 * 10  # 10: bounds the other factors' size
    for g, r in zip(parts(got)[1], parts(ref)[1]):
        assert np.all(np.isfinite(g)) and np.abs(g - r).max() <= small
