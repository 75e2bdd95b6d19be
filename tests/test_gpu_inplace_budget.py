"""Device memory of many small single-buffer handles: the second buffers that such
handles keep are bounded in total and given back."""
import pytest
import torch

from paper_2602_14667_amd import inputs

pytestmark = pytest.mark.gpu

NX, NY, COUNT = 900, 880, 48
STATE = 19 * 4 * 960 * NY  # FP32 rows padded to a multiple of 256 bytes


def used():
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def solver():
    from paper_2602_14667_amd import rrmhd
    return rrmhd.Solver(NX, NY, 0.56, 0.61, inplace=True)


def test_second_buffers_are_bounded_and_given_back():
    print("[gpu] single-buffer budget", flush=True)
    solver().close()  # whatever the first handle of a process allocates
    base = used()
    handles = [solver() for _ in range(COUNT)]
    # allocations come in pieces of a few MiB at most
    assert used() - base <= COUNT * (STATE + (8 << 20)) + (1 << 30)
    u, b = (torch.from_numpy(x).cuda() for x in inputs.random_modes(NX, NY, 0.04, seed=3))
    out = []
    for h in (handles[0], handles[-1]):  # with a second buffer, and without
        h.init(u, b)
        h.step(9)
        out.append(h.moments())
    for x, y in zip(*out):
        assert torch.equal(x, y)
    for h in handles:
        h.close()
    before = used()
    h = solver()
    assert used() - before >= 2 * STATE
    h.close()
