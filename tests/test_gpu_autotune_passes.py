"""What the autotuner keeps about several steps per pass: only entries of a handle
that steps alike are shared, passes are timed whole, and the tuned shape stays in
force for the steps that no pass takes."""
import json

import pytest
import torch

pytestmark = pytest.mark.gpu


def solver(nx, ny, **kw):
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] autotune {nx}x{ny} {kw}", flush=True)
    return rrmhd.Solver(nx, ny, 0.56, 0.61, **kw)


def entries(path):
    return json.loads(path.read_text())


@pytest.mark.parametrize("first", [{"walls": True}, {"force": (1e-6, 0.0)}, {"storage": "f16sr"},
                                   {"equilibrium": "full_maxwell"}])
def test_entry_of_another_kind_of_step_is_not_taken(tmp_path, first):
    """The first handle's plan has no passes, or others than the plain one's."""
    cache = tmp_path / "tune.json"
    n = 700
    layout = {"layout": "planar"}  # as with walls
    a = solver(n, n, **{"storage": "f16", **first, **({} if "walls" in first else layout)})
    a.autotune(str(cache), trials=2)
    b = solver(n, n, storage="f16", **layout)
    b.autotune(str(cache), trials=2)
    assert len(entries(cache)) == 2
    a.close()
    b.close()


def test_earlier_entry_does_not_turn_passes_off(tmp_path):
    """One that was written before passes were timed."""
    cache = tmp_path / "tune.json"
    s = solver(96, 96)
    s.autotune(str(cache), trials=2)
    key, = entries(cache)
    old = key.replace("/passes/", "/")
    entry = {k: v for k, v in entries(cache)[key].items() if k != "multi"}
    cache.write_text(json.dumps({old: entry}))
    s.autotune(str(cache), trials=2)
    new = entries(cache)
    assert any(e.get("multi") == 1 and e["ms"] > 0 for k, e in new.items() if k != old), new
    s.close()


@pytest.mark.parametrize("trials", [1, 3])
@pytest.mark.parametrize("kw", [{}, {"inplace": True}])
def test_few_trials_time_whole_passes(tmp_path, kw, trials):
    """64^2: passes of seven steps against single steps, 1.2 us to 3.1."""
    cache = tmp_path / "tune.json"
    s = solver(64, 64, **kw)
    s.autotune(str(cache), trials=trials)
    e, = entries(cache).values()
    assert e["multi"] == 1
    s.close()


def test_tuned_shape_and_passes_together(tmp_path):
    cache = tmp_path / "tune.json"
    a = solver(96, 80)
    a.autotune(str(cache), trials=2)
    got = entries(cache)
    e, = got.values()
    e.update(bx=16, by=8, xcd=0, nt=1, multi=1)
    cache.write_text(json.dumps(got))
    g = torch.Generator(device="cuda").manual_seed(1)
    u, b = (0.03 * torch.randn(2, 80, 96, dtype=torch.float64, device="cuda", generator=g)
            for _ in range(2))
    ref = solver(96, 80)
    for s in (a, ref):
        s.init(u, b)
    best = a.autotune(str(cache), trials=2)
    assert (best["bx"], best["by"]) == (16, 8) and a.get_launch()[:2] == (16, 8)
    for n in (1, 9, 12):
        a.step(n)
        ref.step(n)
        for x, y in zip(a.moments(), ref.moments()):
            assert torch.equal(x, y), n
    a.close()
    ref.close()


def test_ensemble_with_few_trials(tmp_path):
    """A 32-node tile form (four steps and more per pass) with three trials."""
    from paper_2602_14667_amd import rrmhd
    print("[gpu] autotune ensemble", flush=True)
    cache = tmp_path / "tune.json"
    shapes = [(96, 96)] * 12
    b = rrmhd.Batch(shapes, [0.56] * 12, [0.6] * 12)
    f = torch.zeros(2, 96, 96, dtype=torch.float64, device="cuda")
    for d in range(12):
        b.init(d, f, f)
    b.autotune(str(cache), trials=3)
    assert [e["multi"] for k, e in entries(cache).items() if "passes" in k] == [1], entries(cache)
    b.close()
