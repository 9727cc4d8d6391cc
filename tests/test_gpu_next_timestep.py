"""The timestep that a step's last sweep takes along, against a pass of its own
over the new state, bit for bit (GPU), where float arithmetic cannot bound a
signal speed by itself: gamma within rounding of one, kinetic energies, cell
widths and densities beyond the float range, sound speeds far below it.  The
cells differ little, so a bound that is low by a few parts in 1e5 loses the
cell that sets the timestep."""
import numpy as np
import pytest

from tests.helpers import FIELDS, to_device, to_device_flat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    from paper_1307_2265_amd import ppm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ppm.lib()
    return ppm


def _gas(shape, seed, gamma, rho, speed, eps, spread, eint=1.0):
    """rho, internal energy eps and an x velocity, each cell's energy off by up to
    `spread`; the stored internal energy is eint of the real one."""
    rng = np.random.default_rng(seed)
    e = eps * (1.0 + spread * rng.uniform(-1.0, 1.0, shape))
    u = np.full(shape, speed)
    z = np.zeros(shape)
    return dict(zip(FIELDS, [np.full(shape, rho), u, z, z.copy(), e + 0.5 * u * u, eint * e]))


# gamma, density, x speed, internal energy, its spread, eint's share, cell width, floors
CASES = {
    "gamma 1.0005": (1.0005, 1.0, 0.0, 1.0, 1e-5, 1.0, 0.01, 1e-20),
    "gamma 1.00007": (1.00007, 1.0, 0.0, 1.0, 1e-5, 1.0, 0.01, 1e-20),
    "gamma 1.000001": (1.000001, 1.0, 0.0, 1.0, 1e-3, 1.0, 0.01, 1e-20),
    "gamma 1 + 1e-9": (1.0 + 1e-9, 1.0, 0.0, 1.0, 1e-3, 1.0, 0.01, 1e-20),
    "speed 1e20": (5 / 3, 1.0, 1e20, 1e38, 0.2, 0.5, 0.01, 1e-20),
    "speed 2e19, energy a float": (5 / 3, 1.0, 2e19, 4e36, 0.2, 0.5, 0.01, 1e-20),
    "speed 1e60": (1.4, 1.0, 1e60, 1e118, 0.2, 0.5, 0.01, 1e-20),
    "width 1e39": (5 / 3, 1.0, 0.1, 1.0, 0.1, 1.0, 1e39, 1e-20),
    "width 1e-40": (5 / 3, 1.0, 0.1, 1.0, 0.1, 1.0, 1e-40, 1e-20),
    "density 1e40 at the pressure floor": (5 / 3, 1e40, 0.0, 1e-6, 0.1, 1.0, 0.01, 1e35),
    "energy 1e-50": (5 / 3, 1e20, 0.0, 1e-50, 0.1, 1.0, 0.01, 1e-100),
}
MIXED = ["gamma 1.0005", "gamma 1.00007", "gamma 1.000001", "gamma 1 + 1e-9", "width 1e39",
         "width 1e-40"]


def _check(P, plan, dx, u, c, order):
    import torch
    dt = torch.full((1,), 0.05 * dx / (u + 3.0 * c), dtype=torch.float64, device="cuda")
    want = torch.zeros_like(dt)
    for s in (order, 1 - order):
        plan.ppm_fill_periodic()
        plan.ppm_step_cfl(dt, s)
        plan.ppm_cfl_dt(want)
        assert 0.0 < float(want.item()) < np.inf
        assert float(dt.item()) == float(want.item())
    plan.close()


@pytest.mark.parametrize("name,prec", [(n, "fp64") for n in CASES] + [(n, "mixed") for n in MIXED])
@pytest.mark.parametrize("tiles", [None, "lanes=0", "lanes=0 split=0"])
def test_one_patch(P, name, prec, tiles):
    gamma, rho, u, eps, spread, eint, dx, floor = CASES[name]
    pr = P.PPM_FP64 if prec == "fp64" else P.PPM_MIXED
    shape = tuple(n + 6 for n in (22, 26, 40))
    d = _gas(shape, 11, gamma, rho, u, eps, spread, eint)
    if floor == 1e35:  # the floor sets every pressure, the density the sound speeds
        d["rho"] *= 1.0 + 0.1 * np.random.default_rng(12).uniform(-1.0, 1.0, shape)
    c = np.sqrt(max(gamma * (gamma - 1.0) * eps, gamma * floor / rho))
    patch = to_device(d, pr, dx=(dx, 2.0 * dx, 0.5 * dx))
    prm = P.params(gamma=gamma, p_floor=floor, e_floor=min(1e-20, 1e-3 * eps))
    plan = P.Plan([patch], 1, pr, prm, tile_config=tiles)
    _check(P, plan, 0.5 * dx, u, c, 0)


@pytest.mark.parametrize("tiles", [None, "lanes=1", "persistent=1"])
@pytest.mark.parametrize("name", ["gamma 1.00007", "speed 1e20", "width 1e39"])
def test_several_patches(P, name, tiles):
    gamma, rho, u, eps, spread, eint, dx, floor = CASES[name]
    shapes = [tuple(n + 6 for n in s) for s in ((9, 17, 30), (20, 8, 11), (16, 16, 16))]
    fields = [_gas(s, 21 + i, gamma, rho, u, eps, spread, eint) for i, s in enumerate(shapes)]
    patches = to_device_flat(fields, P.PPM_FP64, [(dx, dx, dx)] * 3, [0] * 3)
    c = np.sqrt(gamma * (gamma - 1.0) * eps)
    prm = P.params(gamma=gamma, p_floor=floor)
    _check(P, P.Plan(patches, 1, P.PPM_FP64, prm, tile_config=tiles), dx, u, c, 1)
