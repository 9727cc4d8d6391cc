"""One persistent launch over several patches (persistent=1): its builds with
HLLC, the diffusive flux, gravity under per-level expansion factors, and the
mixed precision, with every split of the axes between marched and lane-parallel
sweeps (GPU).  FP64 against the oracle, the mixed precision against per-sweep
launches, fields, registers, event counts and the next timesteps bit for bit."""
import numpy as np
import pytest

from paper_1307_2265_amd import workloads as W
from tests.helpers import FIELDS, from_device, oracle_grid
from tests.test_gpu_sources import EXPAND7, _batch_with_sources

pytestmark = pytest.mark.gpu

TILES = ["persistent=1", "persistent=1 lanes=0 batch_block=64", "persistent=1 lanes=7",
         "persistent=1 lanes=2 batch_blocks=3"]
PHYSICS = {"two-shock": 0, "hllc": 16, "diffusion": 32, "sources": 0}  # flags beyond the default


@pytest.fixture(scope="module")
def P():
    import torch
    from paper_1307_2265_amd import ppm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ppm.lib()
    return ppm


def _run(P, prec, physics, tiles, specs, seed):
    """Two steps with the next timestep; the input, the accelerations, the patches,
    the timesteps used and left, the event counts."""
    import torch
    nlev = 7
    fields, accs, patches = _batch_with_sources(P, prec, specs, seed, tiles)
    expand = None
    if physics == "sources":
        expand = torch.tensor([v for av in EXPAND7 for v in av], dtype=torch.float64,
                              device="cuda")
    else:
        for p in patches:
            p.accel = None
    prm = P.params(flags=P.PPM_ALL_FLAGS | PHYSICS[physics])
    plan = P.Plan(patches, nlev, prec, prm, tile_config=tiles)
    if expand is not None:
        plan.ppm_set_expansion(expand)
    dt = torch.zeros(nlev, dtype=torch.float64, device="cuda")
    plan.ppm_cfl_dt(dt)
    dts = [dt.cpu().numpy()]
    for s in range(2):
        plan.ppm_step_cfl(dt, s)
        dts.append(dt.cpu().numpy())
    counts = plan.ppm_event_counts()
    plan.close()
    return fields, accs, patches, dts, counts


@pytest.mark.parametrize("tiles", TILES)
@pytest.mark.parametrize("physics", ["hllc", "diffusion", "sources"])
def test_fp64_equals_oracle(P, O, physics, tiles):
    specs = W.patch_specs(30, 8100)
    fields, accs, patches, dts, counts = _run(P, P.PPM_FP64, physics, tiles, specs, 8200)
    flags = O.params().flags | PHYSICS[physics]
    src = physics == "sources"
    prms = [O.params(flags=flags, a=a, adot=ad) if src else O.params(flags=flags)
            for a, ad in EXPAND7]
    grids = [oracle_grid(O, f, dx=(sp.dx,) * 3, with_reg=True) for f, sp in zip(fields, specs)]
    cnt = [0, 0]
    for s in range(3):
        smax = np.zeros(7)
        for G, sp in zip(grids, specs):
            smax[sp.level] = max(smax[sp.level], O.cfl_signal_max(G, prms[sp.level]))
        want = np.array([prms[l].cfl * (prms[l].a if src else 1.0) / smax[l] if smax[l] > 0
                         else np.inf for l in range(7)])
        assert np.array_equal(dts[s], want), s
        if s == 2:
            break
        for G, acc, sp in zip(grids, accs, specs):
            if src:
                G.accel = acc
            c = O.step(G, prms[sp.level], float(want[sp.level]), s)
            cnt[0] += c.fallback_faces
            cnt[1] += c.floored_cells
    assert counts == tuple(cnt)
    act = (slice(3, -3),) * 3
    for i, (p, G) in enumerate(zip(patches, grids)):
        g = from_device(p)
        for f in FIELDS:
            assert np.array_equal(g[f][act], getattr(G, f)[act]), (i, f)
        assert np.array_equal(p.flux_reg.cpu().numpy(), G.flux_reg), i


@pytest.mark.parametrize("tiles", TILES)
@pytest.mark.parametrize("physics", list(PHYSICS))
def test_mixed_equals_per_sweep_launches(P, physics, tiles):
    import torch
    specs = W.patch_specs(30, 8300)
    _, _, a, dta, ca = _run(P, P.PPM_MIXED, physics, tiles, specs, 8400)
    _, _, b, dtb, cb = _run(P, P.PPM_MIXED, physics, "persistent=0 lanes=1 group=0", specs, 8400)
    assert ca == cb
    assert all(np.array_equal(x, y) for x, y in zip(dta, dtb))
    for i, (p, q) in enumerate(zip(a, b)):
        for f in FIELDS:
            assert torch.equal(getattr(p, f), getattr(q, f)), (i, f)
        assert torch.equal(p.flux_reg, q.flux_reg), i
