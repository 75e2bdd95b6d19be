"""The number of passes that a run of steps takes, and the benchmark's roofline,
which prices the state read and written once per pass."""
from types import SimpleNamespace

import pytest
import torch

from paper_2602_14667_amd import inputs

pytestmark = pytest.mark.gpu


def test_passes_follow_the_handle():
    from paper_2602_14667_amd import rrmhd
    print("[gpu] step passes", flush=True)
    s = rrmhd.Solver(900, 800, 0.56, 0.61)  # marching: four steps per pass
    assert [s.step_passes(n) for n in (0, 1, 4, 6, 40)] == [0, 1, 1, 2, 10]
    s.set_graph_chunk(6)
    assert s.step_passes(12) == 4 and s.step_passes(13) == 5
    s.set_launch(64, 1, 1, 0, 1)
    assert s.step_passes(12) == 12
    s.close()
    s = rrmhd.Solver(64, 64, 0.56, 0.61, inplace=True)  # seven in a tile
    assert s.step_passes(7) == 1 and s.step_passes(8) == 2
    s.close()
    b = rrmhd.Batch([(64, 64)], [0.56], [0.6])
    n, wg = b.step_passes(14)
    assert n == 2 and wg > 0
    b.set_shape(-1, 32, 0, -1)
    assert b.step_passes(14) == (14, b.info()["grid"])
    b.close()


@pytest.mark.parametrize("n,storage", [(256, "f32"), (256, "f16sr"), (1024, "f32")])
def test_turbulence_roofline_counts_launches(n, storage):
    import bench
    from paper_2602_14667_amd import rrmhd
    print(f"[gpu] bench leg {n} {storage}", flush=True)
    fields = tuple(torch.from_numpy(x).cuda() for x in inputs.turbulence(n, 0.04))
    args = SimpleNamespace(n=n, tau=0.52, steps=20, warmup=4, equilibrium="algorithm",
                           inplace=False)
    leg = bench.time_turbulence_leg(torch, rrmhd, args, fields, storage)
    s = rrmhd.Solver(n, n, 0.52, 0.52, storage=storage)
    launches = s.step_passes(20)
    s.close()
    assert launches < 20
    r = leg["roofline"]
    assert r["steps_per_launch"] == pytest.approx(20 / launches, abs=1e-3)
    want = bench.BYTES_PER_NODE[storage] * leg["value"] * 1e6 * (launches / 20) / 1e9
    assert r["achieved"] == pytest.approx(want, rel=1e-2)


def test_tuned_ensemble_leg_counts_launches(monkeypatch):
    """Tuned or not: a shape that was set takes one step per launch."""
    import bench
    from paper_2602_14667_amd import rrmhd
    print("[gpu] bench ensemble leg", flush=True)
    small = inputs.batch_domains(4, seed=0)
    fake = SimpleNamespace(batch_domains=lambda n, seed: small, batch_fields=inputs.batch_fields)
    monkeypatch.setattr(rrmhd.Batch, "autotune",
                        lambda self, path, trials: self.set_shape(-1, 32, 0, -1))
    leg = bench.time_batch_leg(torch, rrmhd, fake, 100, True, False)
    assert leg["roofline"]["steps_per_launch"] == 1
    leg = bench.time_batch_leg(torch, rrmhd, fake, 100, False, False)
    assert leg["roofline"]["steps_per_launch"] > 1
    assert leg["config"]["workgroups_per_launch"] < leg["config"]["tiles"]
