"""ppm_step_cfl_noalloc on patches with enough pencils that sweeps march (GPU):
whole rounds of one marching block per compute unit, a little and a third of a
round past them (the tail launch), one patch and several, both precisions,
against a plan that sweeps every axis lane-parallel, bit for bit.  The patches
are thin, so that a sweep marches pencils by the ten thousands of few cells."""
import pytest

from paper_1307_2265_amd import workloads as W
from tests.helpers import FIELDS, stored_inputs, to_device

pytestmark = pytest.mark.gpu

# patches and sweep order: the thin axis is swept first, where its pencils are most
CASES = {
    "y, below a round": ([(230, 2, 232)], 3),
    "y, a round and 512 pencils": ([(250, 3, 252)], 4),
    "y, a round and a third": ([(290, 1, 290)], 3),
    "y, two rounds and a little": ([(358, 2, 356)], 4),
    "z, below a round": ([(240, 236, 2)], 1),
    "z, a round and 512 pencils": ([(250, 252, 3)], 5),
    "z, a round and a third": ([(290, 290, 1)], 5),
    "y, two patches": ([(240, 2, 238), (230, 3, 250)], 3),
    "z, three patches": ([(240, 230, 2), (200, 250, 1), (9, 7, 11)], 1),
}


@pytest.fixture(scope="module")
def P():
    import torch
    from paper_1307_2265_amd import ppm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ppm.lib()
    return ppm


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("name", list(CASES))
def test_equals_a_lane_parallel_plan(P, name, prec):
    import torch
    pr = P.PPM_FP64 if prec == "fp64" else P.PPM_MIXED
    dims, order = CASES[name]
    inputs = [stored_inputs(W.random_grid(*d, 9100 + i, W.SHOCKED), pr)
              for i, d in enumerate(dims)]
    ref, mine = ([to_device(d, pr, dx=(0.01, 0.02, 0.04), with_reg=True) for d in inputs]
                 for _ in range(2))
    prm = P.params()
    plan = P.Plan(ref, 1, pr, prm, tile_config="lanes=7")
    want = torch.zeros(1, dtype=torch.float64, device="cuda")
    plan.ppm_fill_periodic()
    plan.ppm_cfl_dt(want)
    plan.ppm_step_cfl(want, order)
    dt = torch.full((1,), -1.0, dtype=torch.float64, device="cuda")
    events = P.ppm_step_cfl_noalloc(mine, 1, pr, prm, dt, order,
                                    P.PPM_NOALLOC_FILL | P.PPM_NOALLOC_CFL, events=True)
    assert events == plan.ppm_event_counts()
    assert float(dt.item()) == float(want.item())
    for i, (a, b) in enumerate(zip(mine, ref)):
        for f in FIELDS:
            assert torch.equal(getattr(a, f), getattr(b, f)), (i, f)
        assert torch.equal(a.flux_reg, b.flux_reg), i
    plan.close()
