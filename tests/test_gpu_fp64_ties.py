"""Double quotients, roots and wave-speed reciprocals whose exact values lie
closest to the middle between two doubles (GPU), against IEEE arithmetic and
the oracle, bit for bit.  Roots of 1 + k ulp and reciprocals of 1 - k ulp come
within k^2 2^-106 of such a middle, and gas of sound speed one with a few ulps
of disturbance meets both on every face."""
import numpy as np
import pytest

from paper_1307_2265_amd import workloads as W
from tests.helpers import FIELDS, from_device, oracle_grid, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    from paper_1307_2265_amd import ppm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ppm.lib()
    return ppm


@pytest.mark.parametrize("centre", [1.0, 2.0, 0.25, 1.5, 1.4, 1 / 1.4, 0.1])
def test_quotients_and_roots_around_a_centre(P, centre):
    import torch
    k = np.arange(-5000, 5001)
    b = (np.float64(centre).view(np.int64) + k).view(np.float64)
    for a in (1.0, 1.5, 1.4, centre, 3.0):
        tb = torch.from_numpy(b).cuda()
        tr = torch.from_numpy(b[::-1].copy() if a == centre else np.full_like(b, a)).cuda()
        quot, root = torch.empty_like(tb), torch.empty_like(tb)
        P.ppm_fp64_ops(tr, tb, quot, root)
        assert np.array_equal(quot.cpu().numpy(), tr.cpu().numpy() / b)
        P.ppm_fp64_ops(tb, tr, quot, root)
        assert np.array_equal(root.cpu().numpy(), np.sqrt(b))


@pytest.mark.parametrize("gamma", [1.4, 5.0 / 3.0])
@pytest.mark.parametrize("ulps", [1, 4, 60])
def test_near_uniform_gas_of_unit_sound_speed(P, O, gamma, ulps):
    import torch
    g, n = 3, (70, 9, 11)  # lane-parallel x, marched y and z
    rng = np.random.default_rng(31 + ulps)
    shape = tuple(m + 2 * g for m in n[::-1])
    near = lambda: 1.0 - rng.integers(-ulps, ulps + 1, shape) * 2.0 ** -53
    small = lambda: rng.integers(-ulps, ulps + 1, shape) * 2.0 ** -53
    st = W.stored_from_primitive(near(), small(), small(), small(), near() / gamma, gamma)
    d = dict(zip(FIELDS, [np.ascontiguousarray(a) for a in st]))
    prm, oprm = P.params(gamma=gamma), O.params(gamma=gamma)
    q = to_device(d, P.PPM_FP64, dx=(0.01, 0.01, 0.01), ghost=g)
    grid = oracle_grid(O, d, dx=(0.01, 0.01, 0.01), ghost=g)
    plan = P.Plan([q], 1, P.PPM_FP64, prm, tile_config="lanes=1")
    dt = torch.full((1,), 0.004, dtype=torch.float64, device="cuda")
    for step in range(2):
        plan.ppm_fill_periodic()
        plan.ppm_step(dt, step % 2)
        O.fill_periodic(grid)
        O.step(grid, oprm, 0.004, step % 2)
    got = from_device(q)
    for f in FIELDS:
        assert np.array_equal(got[f], getattr(grid, f)), f
    plan.close()
