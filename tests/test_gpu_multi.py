"""Several steps per launch (LDS tiles and marching strips) against the one-step
kernels, bit for bit: a handle whose launch shape was set explicitly takes one
step per launch.  Sizes sit at the edges of the launch rule's forms: tiles of
16 and 32 nodes, one and several tiles per CU, windows and strips with
remainders, grids narrower than a window and strips that end inside one.
"""
import numpy as np
import pytest
import torch

from paper_2602_14667_amd import inputs

pytestmark = pytest.mark.gpu


def state(s):
    torch.cuda.synchronize()
    out = torch.empty(s.state_bytes(), dtype=torch.uint8, device="cuda")
    s.save_state(out)
    torch.cuda.synchronize()
    return out


def pair(nx, ny, storage, **kw):
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] multi-step {nx}x{ny} {storage} {kw}", flush=True)
    rng = np.random.default_rng(nx * 7919 + ny)
    u = torch.from_numpy(0.03 * rng.standard_normal((2, ny, nx))).cuda()
    b = torch.from_numpy(0.03 * rng.standard_normal((2, ny, nx))).cuda()
    got, ref = (rrmhd.Solver(nx, ny, 0.56, 0.61, storage=storage, **kw) for _ in range(2))
    ref.set_launch(64, 1, 1, 0, 1)
    for s in (got, ref):
        s.init(u, b)
    return got, ref


def check(got, ref, counts):
    for n in counts:
        got.step(n)
        ref.step(n)
        assert got.step_count == ref.step_count
        assert torch.equal(state(got), state(ref)), n
    got.close()
    ref.close()


TILES = [(1, 1), (2, 3), (7, 5), (8, 9), (64, 64), (127, 129), (128, 128), (129, 120), (203, 180),
         (224, 224), (225, 224), (300, 290), (352, 384), (400, 416), (512, 500), (33, 6001)]
MARCH = [(800, 700), (1001, 777), (56, 9000), (57, 9000), (112, 4001), (113, 6000), (224, 2500),
         (225, 2500), (6000, 200), (2048, 1024)]


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape", TILES + MARCH)
def test_periodic_grids_equal_single_steps(shape, storage):
    check(*pair(*shape, storage), [1, 2, 3, 4, 5, 6, 9, 11])


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("force", [(0.0, 0.0), (1e-6, 2e-6)])
@pytest.mark.parametrize("shape", [(1, 2), (5, 3), (64, 64), (130, 33), (200, 190), (512, 256),
                                   (700, 640)])
def test_walls_and_force_equal_single_steps(shape, storage, force):
    check(*pair(*shape, storage, walls=True, force=force, b_wall=(0.001, 0.02)),
          [2, 3, 5, 7, 10])


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(64, 64), (200, 200), (300, 300)])
def test_periodic_force_equals_single_steps(shape, storage):
    check(*pair(*shape, storage, force=(1e-6, -1e-6)), [2, 4, 5, 9])


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("shape", [(64, 64), (65, 64), (96, 97), (256, 256), (257, 256), (353, 351),
                                   (416, 400), (106, 2594), (67, 3001)])
def test_step_counts_of_one_round_tiles(shape, walls, storage):
    """Grids on either side of where a pass of 5 .. 9 steps stops being one
    round of tiles, with step counts that leave uneven passes."""
    check(*pair(*shape, storage, walls=walls), [7, 8, 9, 10, 17, 19])


@pytest.mark.parametrize("kw", [{}, {"walls": True, "b_wall": (0.001, 0.02)}, {"inplace": True},
                                {"force": (1e-6, 2e-6)}, {"codec_scale": 4.0}])
@pytest.mark.parametrize("shape", [(1, 3), (64, 64), (97, 101), (256, 250), (353, 351)])
def test_stochastic_rounding_equals_single_steps(shape, kw):
    """The random bits of every step, node and plane inside a pass."""
    check(*pair(*shape, "f16sr", **kw), [1, 2, 7, 9, 13])


@pytest.mark.parametrize("force", [(0.0, 0.0), (1e-6, 2e-6)])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("shape", [(1300, 1111), (3001, 700)])
def test_many_tiles_per_cu(shape, walls, force):
    check(*pair(*shape, "f32", walls=walls, force=force), [4, 5, 9])


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("shape", [(1, 3), (64, 64), (250, 130), (800, 700)])
def test_small_single_buffer_handles(shape, walls, storage):
    """Single-buffer handles below the size that keeps a second buffer, from
    either phase, either buffer, after a load and around graph replays,
    against the alternating one-step kernels."""
    got, ref = pair(*shape, storage, walls=walls, inplace=True)
    check_steps(got, ref, [1, 4, 5, 9, 1, 1, 3, 2, 7])
    s = state(ref)
    for h in (got, ref):
        h.load_state(s, 40)
    check_steps(got, ref, [5, 1])
    for chunk in (3, 0, 3):
        got.set_graph_chunk(chunk)
        check_steps(got, ref, [7, 6, 5])
    got.close()
    ref.close()


@pytest.mark.parametrize("shape,n,kw", [((64, 64), 10, {}), ((200, 190), 4, {}),
                                        ((200, 190), 16, {"walls": True}), ((900, 800), 4, {}),
                                        ((900, 800), 6, {}), ((200, 190), 4, {"inplace": True})])
def test_steps_recorded_by_the_caller_replay(shape, n, kw):
    """An even number of steps recorded into a caller's graph continues from
    where its last replay ended, with eager steps in between."""
    from paper_2602_14667_amd import rrmhd
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        got, ref = pair(*shape, "f32", **kw)
        both = [(got, ref)]
        batches = [rrmhd.Batch([shape, (70, 40)], [0.55, 0.6], [0.6, 0.55]) for _ in range(2)]
        if not kw:
            batches[1].set_shape(-1, 32, 0, -1)
            for d, (nx, ny) in enumerate([shape, (70, 40)]):
                u, b = (0.02 * torch.randn(2, ny, nx, dtype=torch.float64, device="cuda")
                        for _ in range(2))
                for h in batches:
                    h.init(d, u, b)
            both.append(tuple(batches))
        for g, r in both:
            g.step(2 * n)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=st):
                g.step(n)
            for k in range(3):
                graph.replay()
                torch.cuda.synchronize()
            g.step(2)
            r.step(5 * n + 2)
            fields = (lambda h: [h.moments(d) for d in range(2)]) if g is batches[0] else \
                (lambda h: [h.moments()])
            for a, c in zip(fields(g), fields(r)):
                for x, y in zip(a, c):
                    assert torch.equal(x, y)
            torch.cuda.synchronize()
            g.close()
            r.close()


def check_steps(got, ref, counts):
    for n in counts:
        got.step(n)
        ref.step(n)
        assert got.step_count == ref.step_count
        assert torch.equal(state(got), state(ref)), n


@pytest.mark.parametrize("shape", [(100, 90), (1001, 640)])
def test_planar_layout_scale_and_graph(shape):
    check(*pair(*shape, "f32", layout="planar"), [5, 6])
    check(*pair(*shape, "f16", codec_scale=4.0), [5, 6])
    got, ref = pair(*shape, "f32")
    got.set_graph_chunk(7)  # two launches or three, so replays may end in either buffer
    for k in range(3):
        check_graph(got, ref, 23 + k)
    got.close()
    ref.close()


def check_graph(got, ref, n):
    got.step(n)
    ref.step(n)
    assert torch.equal(state(got), state(ref)), n


def test_nonfinite_values_spread_as_in_single_steps():
    """A NaN and an infinity in the state reach the same nodes either way."""
    for shape in ((96, 80), (900, 800)):
        got, ref = pair(*shape, "f32")
        s = state(ref).view(torch.float32).clone()
        s[5 * shape[0] * shape[1] + 37] = float("nan")
        s[2 * shape[0] * shape[1] + 20 * shape[0] + 11] = float("inf")
        for h in (got, ref):
            h.load_state(s.view(torch.uint8), 0)
            h.step(5)
        a, b = state(got).view(torch.int32), state(ref).view(torch.int32)
        fa, fb = a.view(torch.float32), b.view(torch.float32)
        assert torch.equal(torch.isnan(fa), torch.isnan(fb))
        assert torch.equal(a[~torch.isnan(fa)], b[~torch.isnan(fb)])
        got.close()
        ref.close()


ENSEMBLES = [[(1, 1), (2, 3), (64, 64)], [(64, 40), (24, 24)], [(96, 96), (65, 80)],
             [(256, 129), (96, 100)], [(96, 64), (33, 70), (160, 96)],
             [(224, 225), (130, 64), (64, 190)], [(400, 300), (96, 96), (57, 211)],
             [(1024, 640), (64, 64), (113, 700), (56, 40), (7, 900)],
             [(448, 448)] * 9 + [(225, 31)]]


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("shapes", ENSEMBLES)
def test_ensembles_equal_single_steps(shapes, storage):
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] multi-step ensemble {shapes[:3]} x {len(shapes)} {storage}", flush=True)
    tf = [0.55 + 0.005 * k for k in range(len(shapes))]
    tm = [0.6 - 0.004 * k for k in range(len(shapes))]
    got, ref = (rrmhd.Batch(shapes, tf, tm, storage=storage) for _ in range(2))
    ref.set_shape(-1, 32, 0, -1)  # one step per launch
    rng = np.random.default_rng(len(shapes))
    for d, (nx, ny) in enumerate(shapes):
        u, b = (torch.from_numpy(0.03 * rng.standard_normal((2, ny, nx))).cuda() for _ in range(2))
        for h in (got, ref):
            h.init(d, u, b)
    for k, n in enumerate([1, 2, 3, 4, 5, 9, 23, 24]):
        if k == 6:
            got.set_graph_chunk(7)
        got.step(n)
        ref.step(n)
        assert got.info()["steps"] == ref.info()["steps"]
        for d in range(len(shapes)):
            for a, c in zip(got.moments(d), ref.moments(d)):
                assert torch.equal(a, c), (n, d)
    got.close()
    ref.close()
