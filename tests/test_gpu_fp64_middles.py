"""Double square roots whose exact values lie nearest to the middle between two
doubles, and the reciprocals that start from them, against IEEE arithmetic, bit
for bit (GPU): a refinement that is short of a few bits, or errs to one side,
shows there and nowhere else.  The roots, on both sides of a middle, come from
m^2 + m + c = 0 modulo 2^52 or 2^53."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    from paper_1307_2265_amd import ppm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ppm.lib()
    return ppm


def _recips(P, a, b):
    import torch
    a, b = (torch.from_numpy(np.ascontiguousarray(v, dtype=np.float64)).cuda() for v in (a, b))
    out = torch.empty(5 * a.numel(), dtype=torch.float64, device="cuda")
    P.ppm_fp64_recips(a, b, out)
    return out.cpu().numpy().reshape(5, -1)


def _ops(P, a, b):
    import torch
    a, b = (torch.from_numpy(np.ascontiguousarray(v, dtype=np.float64)).cuda() for v in (a, b))
    quot, root = torch.empty_like(a), torch.empty_like(a)
    P.ppm_fp64_ops(a, b, quot, root)
    return quot.cpu().numpy(), root.cpu().numpy()


def _roots_nearest_middles(cmax):
    """x in [1, 4) with sqrt(x) = (m + 1/2) 2^-52 to within |c| 2^-105."""
    out = []
    for c in range(-cmax, cmax + 1, 2):
        for k, lo, hi in ((52, 2 ** 52, int(2 ** 52.5)), (53, int(2 ** 52.5), 2 ** 53)):
            t, r = 1 - 4 * c, 1  # (2m + 1)^2 = 1 - 4c modulo 2^(k+2): a root, bit by bit
            for i in range(3, k + 2):
                if (r * r - t) >> i & 1:
                    r += 1 << (i - 1)
            for s in {q % 2 ** (k + 2) for q in (r, -r, r + 2 ** (k + 1), -r + 2 ** (k + 1))}:
                for m in ((s - 1) // 2, (s - 1) // 2 + 2 ** (k + 1)):
                    x, rest = divmod(m * m + m + c, 2 ** k)
                    if lo <= m < hi and rest == 0 and 2 ** 52 <= x < 2 ** 53:
                        out.append(float(x) * 2.0 ** (k - 104))
    return np.array(sorted(set(out)))


@pytest.mark.parametrize("scale", [1.0, 4.0, 2.0 ** 80, 2.0 ** -600])
def test_roots_nearest_middles(P, scale):
    x = _roots_nearest_middles(400) * scale
    assert x.size > 500
    assert np.array_equal(_ops(P, x, x)[1], np.sqrt(x))
    o = _recips(P, x, x[::-1].copy())
    assert np.array_equal(o[0], np.sqrt(x))
    assert np.array_equal(o[1], 1.0 / np.sqrt(x))
    assert np.array_equal(o[3], np.sqrt(x) * np.sqrt(x[::-1]))
    assert np.array_equal(o[4], 1.0 / o[3])


def test_empty_and_invalid_calls(P):
    import torch
    z = torch.empty(0, dtype=torch.float64, device="cuda")
    P.ppm_fp64_recips(z, z, z)
    L = P.lib()
    assert L.ppm_fp64_recips(None, None, None, 5, None) == P.PPM_EINVAL
    assert L.ppm_fp64_recips(None, None, None, -1, None) == P.PPM_EINVAL
