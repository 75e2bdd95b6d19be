"""Single-buffer boxes a little past the last-level cache, which take streaming stores
in workgroups of 64 (rows of 64, or planes a power of two apart), against the
two-buffer step, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(64, 160, 160), (128, 128, 128)])
def test_streaming_single_buffer_steps(shape):
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] 3D single-buffer stores {shape}", flush=True)
    nx, ny, nz = shape
    g = torch.Generator(device="cuda").manual_seed(nz)
    u, b = (0.02 * torch.randn(3, nz, ny, nx, dtype=torch.float64, device="cuda", generator=g)
            for _ in range(2))
    one, two = (rrmhd.Solver3D(nx, ny, nz, 0.56, 0.6, inplace=k) for k in (True, False))
    for s in (one, two):
        s.init(u, b)
    for n in (1, 2, 4):
        for s in (one, two):
            s.step(n)
        for x, y in zip(one.moments(), two.moments()):
            assert torch.equal(x, y), n
    one.close()
    two.close()
