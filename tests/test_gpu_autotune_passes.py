"""What the autotuner keeps about several steps per pass: only entries of a handle
that steps alike are shared."""
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
