"""The matrix-core training network at batch sizes around its 16-sample
wavefronts, 64-sample workgroups and 512-workgroup grid, and in the tails of
the GELU, against the FP64 oracle.

Tolerance: a gradient entry is a sum over samples of products that each went
through chains of at most 64 + 64 FP32 multiply-adds and the GELU (a few units
in the last place each), so its relative L2 error stays below 128 * 2^-24 =
7.6e-6; twice that is allowed.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 2 * 128 * 2.0 ** -24


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def f32(a):
    return np.asarray(a, dtype=np.float32).astype(np.float64)


@pytest.mark.parametrize("n,gain", [(1, 1.0), (15, 1.0), (16, 1.0), (17, 1.0), (63, 1.0), (64, 1.0),
                                    (65, 1.0), (32768, 1.0), (32769, 1.0), (40000, 1.0),
                                    (2000, 6.0)])
def test_loss_gradient_at_group_edges(n, gain):
    """gain: scale of the first layer (6: pre-activations far into both tails)."""
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] training network n={n} gain={gain}", flush=True)
    rng = np.random.default_rng(n)
    p = np.zeros(oracle.NPARAM)
    p[0:512] = gain * rng.standard_normal(512) / np.sqrt(8)
    p[512:576] = 0.1 * rng.standard_normal(64)
    p[576:4672] = rng.standard_normal(4096) / np.sqrt(64)
    p[4672:4736] = 0.1 * rng.standard_normal(64)
    p[4736:4928] = rng.standard_normal(192) / np.sqrt(64)
    p[4928:] = 0.1 * rng.standard_normal(3)
    nm = np.concatenate([np.zeros(8), np.ones(8), [1e-4, 2e-4, 1e-4]])
    p, nm = f32(p), f32(nm)
    x = f32(rng.standard_normal((n, 8)))
    t = f32(1e-4 * rng.standard_normal((n, 3)))
    loss_ref, g_ref = oracle.mlp_loss_grad(p, nm, x, t / nm[16:19])
    tr = rrmhd.Trainer(n)
    grad = torch.full((4931,), float("nan"), dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    for _ in range(2):  # a second call on the same workspace gives the same bits
        tr.loss_grad(dev(p), dev(nm), dev(x), dev(t), grad, loss)
        g = grad.cpu().numpy()
        if _:
            assert np.array_equal(g, first)
        first = g
    e = np.linalg.norm(g - g_ref) / np.linalg.norm(g_ref)
    assert e < TOL, e
    assert abs(loss.item() - loss_ref) < TOL * abs(loss_ref)
    tr.close()
