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


@pytest.mark.parametrize("nc,factor", [(1, 2), (15, 2), (16, 4), (17, 4), (16, 8), (33, 8),
                                       (16, 3), (5, 6)])
@pytest.mark.parametrize("skew", [0, 1])
def test_box_filter_factors_and_alignment(nc, factor, skew):
    """Compiled and general factors, fields at 16-byte and at 8-byte bases;
    and den, summed per workgroup first.  FP64 sums of at most 64 values
    (1089 for den): 1e-13 relative to the largest value is over ten times
    their rounding."""
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] box filter nc={nc} factor={factor} skew={skew}", flush=True)
    n = nc * factor
    g = np.random.default_rng(10 * nc + factor)

    def field(*shape):
        a = 0.05 * g.standard_normal(shape) + (1.0 if len(shape) == 2 else 0.0)
        t = torch.empty(a.size + skew, dtype=torch.float64, device="cuda")[skew:].view(shape)
        t.copy_(torch.from_numpy(a))
        return a, t

    def mean(a):
        return a.reshape(nc, factor, nc, factor).mean(axis=(1, 3))

    (r0, tr0), (u0, tu0), (b0, tb0) = field(n, n), field(2, n, n), field(2, n, n)
    (r1, tr1), (u1, tu1), (b1, tb1) = field(n, n), field(2, n, n), field(2, n, n)
    out = rrmhd.train_box_filter(tr0, tu0, tb0, factor).cpu().numpy()
    want = [r0, r0 * u0[0], r0 * u0[1], b0[0], b0[1], r0 * u0[0] ** 2, r0 * u0[0] * u0[1],
            r0 * u0[1] ** 2, 0.5 * (b0[1] ** 2 - b0[0] ** 2), -b0[0] * b0[1]]
    for k, w in enumerate(want):
        assert np.abs(out[k] - mean(w)).max() <= 1e-13 * np.abs(w).max(), k
    _, _, den = rrmhd.train_onestep_samples((tr0, tu0, tb0), (tr1, tu1, tb1), factor, 0.55)
    dj = [mean(r1 * u1[a]) - mean(r0 * u0[a]) for a in range(2)]
    ref = (dj[0] ** 2 + dj[1] ** 2).sum()
    assert abs(den.item() - ref) <= 1e-12 * ref
