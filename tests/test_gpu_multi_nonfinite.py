"""NaN and infinities in the state reach the same nodes in passes of several steps
as in single steps: every storage, walls, force and the ensemble."""
import numpy as np
import pytest
import torch

from test_gpu_multi import pair, state

pytestmark = pytest.mark.gpu


def same(a, b, what):
    assert torch.equal(torch.isnan(a), torch.isnan(b)), what
    bits = {2: torch.int16, 4: torch.int32, 8: torch.int64}[a.element_size()]
    ok = ~torch.isnan(a)
    assert torch.equal(a.view(bits)[ok], b.view(bits)[ok]), what


@pytest.mark.parametrize("shape", [(96, 80), (250, 240), (700, 640)])
@pytest.mark.parametrize("storage", ["f32", "f16", "f16sr"])
@pytest.mark.parametrize("kw", [{}, {"walls": True, "b_wall": (0.001, 0.02)},
                                {"force": (1e-6, 2e-6)},
                                {"walls": True, "force": (1e-6, 0.0)}, {"inplace": True}])
def test_nonfinite_state(shape, storage, kw):
    got, ref = pair(*shape, storage, **kw)
    real = torch.float32 if storage == "f32" else torch.float16
    nx, ny = shape
    s = state(ref).view(real).clone()
    s[5 * nx * ny + 37] = float("nan")             # next to a wall, where there is one
    s[2 * nx * ny + (ny // 2) * nx + 11] = float("inf")
    s[12 * nx * ny + (ny - 3) * nx + nx - 1] = float("-inf")
    for h in (got, ref):
        h.load_state(s.view(torch.uint8), 0)
    for n in (5, 4, 9):
        for h in (got, ref):
            h.step(n)
        same(state(got).view(real), state(ref).view(real), n)
    got.close()
    ref.close()


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shapes", [[(64, 64), (33, 40)], [(256, 129), (96, 100)],
                                    [(1024, 640), (113, 700)]])
def test_nonfinite_ensemble(shapes, storage):
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] non-finite ensemble {shapes} {storage}", flush=True)
    got, ref = (rrmhd.Batch(shapes, [0.56, 0.6], [0.6, 0.56], storage=storage) for _ in range(2))
    ref.set_shape(-1, 32, 0, -1)
    rng = np.random.default_rng(4)
    for d, (nx, ny) in enumerate(shapes):
        u, b = 0.03 * rng.standard_normal((2, 2, ny, nx))
        u[0, ny // 3, 5] = np.nan
        b[1, ny - 1, nx - 2] = np.inf
        for h in (got, ref):
            h.init(d, torch.from_numpy(u).cuda(), torch.from_numpy(b).cuda())
    for n in (5, 4, 9):
        for h in (got, ref):
            h.step(n)
        for d in range(2):
            for x, y in zip(got.moments(d), ref.moments(d)):
                same(x, y, (n, d))
    got.close()
    ref.close()
