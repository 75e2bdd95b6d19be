"""Runs whose length is no whole number of passes, and grids where single steps are
the faster: how many passes they take, and that the bits stay those of single steps."""
import pytest

from test_gpu_multi import check, pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,storage,kw", [
    ((64, 5000), "f16", {"walls": True}), ((64, 5000), "f16", {}), ((64, 3000), "f16", {}),
    ((64, 5000), "f32", {"inplace": True}), ((127, 4000), "f16", {"inplace": True})])
def test_single_steps_where_they_are_faster(shape, storage, kw):
    got, ref = pair(*shape, storage, **kw)
    assert got.step_passes(40) == 40
    check(got, ref, [3])


@pytest.mark.parametrize("shape,storage,kw,passes", [
    ((512, 500), "f32", {}, {5: 1, 6: 2, 7: 3, 8: 2, 10: 2, 11: 3}),  # five steps per pass
    ((512, 500), "f32", {"inplace": True}, {6: 2, 7: 3, 8: 2, 11: 3}),
    ((64, 3000), "f32", {}, {6: 2, 7: 3, 10: 2}),
    ((400, 400), "f32", {"walls": True}, {6: 3, 7: 4, 12: 3})])  # four
def test_uneven_runs_take_full_passes_first(shape, storage, kw, passes):
    got, ref = pair(*shape, storage, **kw)
    assert {n: got.step_passes(n) for n in passes} == passes
    check(got, ref, list(passes))
