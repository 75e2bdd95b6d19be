"""Calls that the caller records into a graph of its own, mixed with direct calls:
whatever is stepped, initialised or loaded between replays, a replay works on the
state as single steps leave it.  The reference takes the same steps one at a time,
without a graph.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


class Grid:
    """A handle on one grid; `single`: one step per launch."""

    def __init__(self, shape, single, **kw):
        from paper_2602_14667_amd import rrmhd
        self.nx, self.ny = shape
        self.h = rrmhd.Solver(self.nx, self.ny, 0.56, 0.61, **kw)
        if single:
            self.h.set_launch(64, 1, 1, 0, 1)

    def init(self, seed):
        rng = np.random.default_rng(seed)
        self.h.init(*(torch.from_numpy(0.03 * rng.standard_normal((2, self.ny, self.nx))).cuda()
                      for _ in range(2)))

    def step(self, n):
        self.h.step(n)

    def fields(self):
        return list(self.h.moments())

    def close(self):
        self.h.close()


class Ensemble(Grid):
    def __init__(self, shape, single, **kw):
        from paper_2602_14667_amd import rrmhd
        self.shapes = [shape, (70, 40)]
        self.h = rrmhd.Batch(self.shapes, [0.55, 0.6], [0.6, 0.55], **kw)
        if single:
            self.h.set_shape(-1, 32, 0, -1)

    def init(self, seed):
        rng = np.random.default_rng(seed)
        for d, (nx, ny) in enumerate(self.shapes):
            self.h.init(d, *(torch.from_numpy(0.03 * rng.standard_normal((2, ny, nx))).cuda()
                             for _ in range(2)))

    def fields(self):
        return [t for d in range(2) for t in self.h.moments(d)]


GRIDS = [(Grid, (64, 64), {}), (Grid, (200, 190), {"walls": True, "storage": "f16"}),
         (Grid, (900, 800), {}), (Grid, (64, 64), {"inplace": True}),
         (Grid, (250, 130), {"inplace": True, "storage": "f16"}),
         (Grid, (900, 800), {"inplace": True})]
ENSEMBLES = [(Ensemble, (64, 64), {}), (Ensemble, (900, 800), {})]


def both(case):
    kind, shape, kw = case
    print(f"[gpu] recorded {kind.__name__} {shape} {kw}", flush=True)
    pair = [kind(shape, single, **kw) for single in (False, True)]
    for h in pair:
        h.init(1)
    return pair


def record(fn, st):
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        out = fn()
    return graph, out


def same(got, want, what):
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b), what


@pytest.mark.parametrize("case", GRIDS + ENSEMBLES)
@pytest.mark.parametrize("n", [2, 4])
@pytest.mark.parametrize("first", [4, 3])
def test_replays_between_direct_steps(case, n, first):
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        got, ref = both(case)
        got.step(first)
        ref.step(first)
        graph, _ = record(lambda: got.step(n), st)
        done = 0
        for e in (0, 2, 4, 10, 1, 3, 16, 7, 5):
            got.step(e)
            ref.step(e)
            done += e
            if done % 2 == 0:  # from where the recorded steps start
                graph.replay()
                ref.step(n)
            same(got.fields(), ref.fields(), (e, done))
        got.close()
        ref.close()


@pytest.mark.parametrize("case", GRIDS)
@pytest.mark.parametrize("load", [False, True])
def test_replay_after_a_new_start(case, load):
    """init and load_state put the state where the recorded steps expect it."""
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        got, ref = both(case)
        for h in (got, ref):
            h.step(4)
        graph, _ = record(lambda: got.step(4), st)
        saved = torch.empty(ref.h.state_bytes(), dtype=torch.uint8, device="cuda")
        ref.step(2)
        ref.h.save_state(saved)
        for k in range(2):
            for h in (got, ref):
                if load:
                    h.h.load_state(saved, 6)
                else:
                    h.init(2 + k)
            graph.replay()
            ref.step(4)
            same(got.fields(), ref.fields(), k)
            for h in (got, ref):
                h.step(6)
            same(got.fields(), ref.fields(), k)
        got.close()
        ref.close()


@pytest.mark.parametrize("case", [c for c in GRIDS if "inplace" in c[2]] + [
    (Grid, (1, 3), {"inplace": True}), (Grid, (64, 64), {"inplace": True, "walls": True}),
    (Grid, (97, 101), {"inplace": True, "walls": True, "b_wall": (0.001, 0.02), "storage": "f16"}),
    (Grid, (64, 64), {"inplace": True, "layout": "planar", "force": (1e-6, 0.0)}),
    (Grid, (97, 60), {"inplace": True, "storage": "f16sr"})])
@pytest.mark.parametrize("first", [7, 4, 1])
def test_one_buffer_replay_in_either_phase(case, first, tmp_path):
    """The phase that the recorded steps start from comes back with the parity of
    the steps, also after a new start and where passes of an odd number of steps
    came before the recording."""
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        got, ref = both(case)
        for h in (got, ref):
            h.step(first)
        graph, _ = record(lambda: got.step(2), st)
        # random bits are keyed by the step number, which a replay keeps
        keyed = case[2].get("storage") == "f16sr"
        saved = torch.empty(ref.h.state_bytes(), dtype=torch.uint8, device="cuda")
        ref.h.save_state(saved)
        ref.h.save(str(tmp_path / "state"))
        starts = [lambda h: h.init(5), lambda h: h.h.load_state(saved, 0),
                  lambda h: h.h.load(str(tmp_path / "state"))]
        for k, start in enumerate(starts):
            for h in (got, ref):
                start(h)
            same(got.fields(), ref.fields(), (k, "start"))
            for h in (got, ref):
                h.step(first % 2 + 2)
            same(got.fields(), ref.fields(), (k, "direct"))
            if not keyed:
                graph.replay()
                ref.step(2)
                same(got.fields(), ref.fields(), (k, "replay"))
            a, b = (torch.empty_like(saved) for _ in range(2))
            got.h.save_state(a)
            ref.h.save_state(b)
            same([a], [b], (k, "state"))
        got.close()
        ref.close()


@pytest.mark.parametrize("case", GRIDS + ENSEMBLES)
def test_recorded_fields_after_direct_steps(case):
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        got, ref = both(case)
        for h in (got, ref):
            h.step(4)
        graph, out = record(got.fields, st)
        for n in (2, 4, 6, 8):
            got.step(n)
            ref.step(n)
            graph.replay()
            same(out, ref.fields(), n)
        got.close()
        ref.close()


@pytest.mark.parametrize("case", GRIDS + ENSEMBLES)
@pytest.mark.parametrize("chunk", [4, 6, 7])
def test_recorded_fields_with_graph_chunks(case, chunk):
    """The handle's own graphs, built before and after the recording."""
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        got, ref = both(case)
        got.h.set_graph_chunk(chunk)
        for h in (got, ref):
            h.step(3 * chunk)
            h.step(chunk + 1)
            h.step(chunk - 1)
        same(got.fields(), ref.fields(), "before")
        graph, out = record(got.fields, st)
        for n in (2 * chunk, 2 * chunk + 2, 4, 4 * chunk):
            got.step(n)
            ref.step(n)
            graph.replay()
            same(out, ref.fields(), n)
            same(got.fields(), ref.fields(), n)
        got.h.set_graph_chunk(0)
        for h in (got, ref):
            h.step(8)
        graph.replay()
        same(out, ref.fields(), "plain")
        got.close()
        ref.close()
