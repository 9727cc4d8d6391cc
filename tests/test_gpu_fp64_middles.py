"""Double reciprocals, quotients and roots whose exact values lie nearest to the
middle between two doubles, against IEEE arithmetic, bit for bit (GPU): a
refinement that is short of a few bits, or errs to one side, shows there and
nowhere else.  Reciprocals on both sides of a middle from the factors of 2^106 + j
(b m = 2^106 + j with m odd, |j| < 1000, one of b = 2^53 - k among them), roots
on both sides from m^2 + m + c = 0 modulo 2^52 or 2^53, quotients by divisors just
below a power of two."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# divisors of 2^106 + j, |j| < 1000: mantissas whose reciprocals lie nearest a middle
RECIPROCALS = np.array([
    0x1ffffff8000001, 0x1c69bf28eba166, 0x181efe51ead722, 0x1fffffffffffff, 0x1ffffffffffffd,
    0x1024a3bd98da02, 0x109107683ee29e, 0x11d3799c32581e, 0x12bf5907e316d2, 0x130a0dd90e13a2,
    0x13a324a526d5ee, 0x14cad5a5fa03ee, 0x163baaac17d1e2, 0x17641c46f799ee, 0x17f52093014f0e,
    0x199e1b447e99c2, 0x1a0b8ffffcbe8e, 0x1b227794e85702, 0x1d5b9032f086be, 0x1de441d5331432,
    0x1e756f08df1792, 0x1014ca35e947b6, 0x10d03f8a57cc76, 0x1125e52b034982, 0x120a8f5bbf2106,
    0x1379cb88f092f2, 0x13d75d54b37492, 0x156a8cb0234262, 0x16026c81a85766, 0x16f0f27bf434d6,
    0x1806c89fcb9452, 0x18401cbcdb5596, 0x1a149bad85de72, 0x1aa7c88ee59082, 0x1c2693dcf34742,
    0x1e8d517d09c5c2, 0x1f65fad23b0d86, 0x10aadc6f562fdc, 0x124936db76db70, 0x1520e032e63b90,
    0x17466b6b56eabd, 0x1711ac1b14466f, 0x10ff1f77807040, 0x12430bb7fc47c0, 0x136c813c26c7c0,
    0x1641955b897cc0, 0x178ce42e018cc0, 0x19bc8339534ac0, 0x1cad73b9a5ddc0, 0x1f363e7064e0c0,
    0x100ea20adff075, 0x1153f6c9b53ff1, 0x171d966c5b3a7c, 0x1cf891f1108b9a, 0x167c3b37149a99,
    0x147ccffff331fe, 0x1ceaf1e08166da, 0x1e198742a280c5, 0x1cb476148c9a8e, 0x1b23765914a5c8,
    0x11ffb0eca57ed1, 0x1750833e9fa280, 0x11c496fa5f98db, 0x17b8e26adb90cb, 0x189793162569d0,
    0x16aed5700794e1, 0x1a45e5c536dec7, 0x1ab82d2eb4e0d9, 0x1864b9872eb4c3, 0x1e5f75270d0440,
    0x147ac10975c71b, 0x17b0ad653f26ad, 0x1041b09fcb63e1, 0x1c9f84ddc08fe8, 0x14c935a5867cc9,
    0x10318c5d4c3036, 0x15fbe3f9c7e621, 0x1f252a51329e9d, 0x12192f0aab2004, 0x15279312de8f82,
    0x16fe6c76318951, 0x143c4c6afeda3b,
], dtype=np.uint64).astype(np.float64) * 2.0 ** -52

# a and k: a / (2^53 - k) lies as near a middle as any quotient, 1 / (2^53 - k)
# within 2^-73 of one
QUOTIENTS = [
    (7724407935011299, 553393847), (7378020231649012, 600239903), (5496123684746194, 615062873),
    (7798113501157545, 615062875), (4971568049184148, 629536921), (8106995195691211, 643685585),
    (8622961980485001, 657529869), (8778620841357299, 671088613), (6924089366212834, 684378787),
    (6228519934250839, 697415743), (5148843966888631, 710213429), (7995315034086201, 722784553),
    (7241516965289050, 722784555), (5935641364162861, 735140739), (4651301520380665, 735140741),
    (8510468517810118, 747292649), (7563203641900492, 759250091), (7044686115017426, 794042751),
    (7683655481748075, 805306329), (6214243195827892, 805306331), (6464141998206034, 816414527),
    (5198710519611577, 827373601), (4862944922901041, 838189401), (5500617519576225, 848867403),
]


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


@pytest.mark.parametrize("scale", [1.0, 0.5, 2.0, 2.0 ** 40, 2.0 ** -300])
def test_reciprocals_nearest_middles(P, scale):
    b = RECIPROCALS * scale
    o = _recips(P, b * b, np.ones_like(b))
    assert np.array_equal(o[0], b)
    assert np.array_equal(o[1], 1.0 / b)
    assert np.array_equal(o[3], b)
    assert np.array_equal(o[4], 1.0 / b)
    assert np.array_equal(_recips(P, b, b)[2], 1.0 / b)
    assert np.array_equal(_ops(P, np.ones_like(b), b)[0], 1.0 / b)


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


def test_quotients_nearest_middles_below_a_power_of_two(P):
    a, b = [], []
    for k in range(1, 2 ** 13, 2):
        d = 2 ** 53 - k
        for p in (53, 54):  # a 2^p = +-1 modulo d
            i = pow(2, -p, d)
            for v in (i, d - i):
                if 2 ** 52 <= v < 2 ** 53:
                    a.append(float(v))
                    b.append(float(d))
    assert len(a) > 4000
    a = np.array(a + [float(v) for v, _ in QUOTIENTS])
    b = np.array(b + [float(2 ** 53 - k) for _, k in QUOTIENTS])
    assert np.array_equal(_ops(P, a, b)[0], a / b)


def test_special_operands_of_the_tracing(P):
    x = np.array([0.0, -0.0, 1.0, 4.0, np.inf, -1.0, -np.inf, np.nan, 1e-232, 1e232, 0.25])
    o = _recips(P, x, np.ones_like(x))
    with np.errstate(divide="ignore", invalid="ignore"):
        root = np.sqrt(x)
        want = [root, 1.0 / root, 1.0 / x]
    for got, w in zip(o, want):
        assert np.array_equal(got, w, equal_nan=True), (got, w)
        assert np.array_equal(np.signbit(got[~np.isnan(w)]), np.signbit(w[~np.isnan(w)]))


def test_empty_and_invalid_calls(P):
    import torch
    z = torch.empty(0, dtype=torch.float64, device="cuda")
    P.ppm_fp64_recips(z, z, z)
    L = P.lib()
    assert L.ppm_fp64_recips(None, None, None, 5, None) == P.PPM_EINVAL
    assert L.ppm_fp64_recips(None, None, None, -1, None) == P.PPM_EINVAL
