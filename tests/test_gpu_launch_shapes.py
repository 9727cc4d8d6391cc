"""The launch shapes a plan chooses against the oracle, bit for bit (GPU):
lane-parallel runs at the edges of their 64-lane segments (one pencil of 64
cells, one more, two segments' 118, one more), few and many pencils per group
of waves, pencils shorter than a segment, the y and z axes at their default
limits' two sides, and several patches with per-sweep launches on every axis
or in one persistent launch.  The FP64 path does the oracle's operations in
the oracle's order whatever the shape, so no difference is allowed."""
import numpy as np
import pytest

from paper_1307_2265_amd import workloads as W
from tests.helpers import FIELDS, from_device, oracle_grid, to_device, to_device_flat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    from paper_1307_2265_amd import ppm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ppm.lib()
    return ppm


def _dt(value=None):
    import torch
    return torch.full((1,), 0.0 if value is None else value, dtype=torch.float64, device="cuda")


# (nx, ny, nz, ghost): active cells; a pencil holds 2 ghost more
ONE_PATCH = [(58, 5, 4, 3), (59, 4, 5, 3), (112, 3, 6, 3), (113, 6, 3, 3), (5, 58, 113, 3),
             (1, 1, 1, 3), (7, 2, 300, 4), (24, 40, 35, 3), (300, 19, 2, 6)]


@pytest.mark.parametrize("dims", ONE_PATCH, ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("tiles", [None, "lanes=7 lanes_block=64"])
def test_one_patch_step_and_timestep(P, O, dims, tiles):
    import torch
    nx, ny, nz, g = dims
    d = W.random_grid(nx, ny, nz, 6100 + nx, W.SHOCKED, ghost=g)
    dx = (0.5, 0.25, 1.0)
    G = oracle_grid(O, d, ghost=g, dx=dx)
    prm = O.params()
    patch = to_device(d, P.PPM_FP64, ghost=g, dx=dx)
    plan = P.Plan([patch], 1, P.PPM_FP64, P.params(), tile_config=tiles)
    dt = _dt()
    plan.ppm_fill_periodic()
    plan.ppm_cfl_dt(dt)
    for s in (0, 1):
        O.fill_periodic(G)
        want = O.cfl_dt(G, prm)
        assert float(dt.item()) == want
        O.step(G, prm, want, s)
        plan.ppm_fill_periodic()
        plan.ppm_step_cfl(dt, s)
    torch.cuda.synchronize()
    out = from_device(patch)
    for f in FIELDS:
        assert np.array_equal(out[f], getattr(G, f)), f
    plan.close()


@pytest.mark.parametrize("npatch", [2, 9, 40])
@pytest.mark.parametrize("tiles", [None, "lanes=1", "lanes=7 lanes_block=256", "persistent=1",
                                   "persistent=1 lanes=7"])
def test_several_patches_step(P, O, npatch, tiles):
    import torch
    rng = np.random.default_rng(77)
    dims = [tuple(int(v) for v in rng.integers(1, 40, 3)) for _ in range(npatch)]
    fields = [W.random_grid(*d, 6300 + i, W.SHOCKED, seeded_ghosts=True)
              for i, d in enumerate(dims)]
    patches = to_device_flat(fields, P.PPM_FP64, [(1.0, 0.5, 0.25)] * npatch, [0] * npatch,
                             with_reg=True)
    plan = P.Plan(patches, 1, P.PPM_FP64, P.params(), tile_config=tiles)
    dt = _dt(2e-3)
    for s in (0, 1):
        plan.ppm_step(dt, s)
    torch.cuda.synchronize()
    prm = O.params()
    for p, f in zip(patches, fields):
        G = oracle_grid(O, f, dx=(1.0, 0.5, 0.25), with_reg=True)
        for s in (0, 1):
            O.step(G, prm, 2e-3, s)
        out = from_device(p)
        for k in FIELDS:
            assert np.array_equal(out[k], getattr(G, k)), k
        assert np.array_equal(p.flux_reg.cpu().numpy(), G.flux_reg)
    plan.close()


@pytest.mark.parametrize("n", [16, 17, 18, 19, 40, 41])
@pytest.mark.parametrize("ghost", [3, 4, 5, 6])
@pytest.mark.parametrize("tiles", ["lanes=0", "lanes=0 split=0"])
def test_marching_by_halves_at_odd_and_even_lengths(P, O, n, ghost, tiles):
    # two iterations to a round: either half of a pencil may end in the middle of
    # one, next to the cells the other half owns; fluxes and event counts too
    import torch
    d = W.random_grid(n, n + 1, n + 2, 6500 + n + ghost, W.SHOCKED, ghost=ghost)
    G = oracle_grid(O, d, ghost=ghost, dx=(1.0, 0.5, 0.25), with_reg=True)
    patch = to_device(d, P.PPM_FP64, ghost=ghost, dx=(1.0, 0.5, 0.25), with_reg=True)
    plan = P.Plan([patch], 1, P.PPM_FP64, P.params(), tile_config=tiles)
    dt = _dt(2e-3)
    fb = fl = 0
    for s in (0, 1):
        O.fill_periodic(G)
        c = O.step(G, O.params(), 2e-3, s)
        fb, fl = fb + c.fallback_faces, fl + c.floored_cells
        plan.ppm_fill_periodic()
        plan.ppm_step(dt, s)
    torch.cuda.synchronize()
    out = from_device(patch)
    for f in FIELDS:
        assert np.array_equal(out[f], getattr(G, f)), f
    assert np.array_equal(patch.flux_reg.cpu().numpy(), G.flux_reg)
    assert plan.ppm_event_counts() == (fb, fl)
    plan.close()


@pytest.mark.parametrize("dims", [(135, 70, 137), (70, 240, 139), (129, 129, 40)])
@pytest.mark.parametrize("tiles", ["lanes=0 block=64", "lanes=1 block=64"])
def test_halves_and_tails_as_a_plan_chooses_them(P, O, dims, tiles):
    # rounds of 64-thread blocks: sweeps of less than one round, of a little and of
    # more than half a round past a whole number of them, by halves and whole
    import torch
    nx, ny, nz = dims
    d = W.random_grid(nx, ny, nz, 6700 + nx, W.SHOCKED)
    dx = (1.0, 0.5, 0.25)
    G = oracle_grid(O, d, dx=dx)
    patch = to_device(d, P.PPM_FP64, dx=dx)
    plan = P.Plan([patch], 1, P.PPM_FP64, P.params(), tile_config=tiles)
    dt = _dt(2e-3)
    for s in (0, 1):
        O.fill_periodic(G)
        O.step(G, O.params(), 2e-3, s)
        want = O.cfl_dt(G, O.params())
        plan.ppm_fill_periodic()
        dt.fill_(2e-3)
        plan.ppm_step_cfl(dt, s)
        assert float(dt.item()) == want
    torch.cuda.synchronize()
    out = from_device(patch)
    for f in FIELDS:
        assert np.array_equal(out[f], getattr(G, f)), f
    plan.close()
