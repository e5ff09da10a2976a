"""The kernels' shortened quotients and roots (vs_device.h: div_rcp, div_by,
half_rsqrt, hom_div) bit for bit against the operators: reciprocal and root over
every float of their ranges on the device, quotients next to rounding midpoints and
projections that leave the shortened form's range against numpy's IEEE operators.
Coverage decisions and the parity of flow, blend and Jacobi steps rest on them."""
import ctypes as C
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

RCP, HALF_RSQRT, OPERATORS = 0, 1, 2


@pytest.fixture(scope="module")
def dm():
    from paper_2308_09209_amd import build as B
    if not os.path.exists(B.MATH_OUT):
        B.build_math()
    return C.CDLL(B.MATH_OUT)


def say(*a):
    print(*a, flush=True)


def cu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def ptr(t):
    return C.c_void_p(t.data_ptr())


def bits(a):
    return np.ascontiguousarray(a, np.float32).view(np.uint32)


def pattern(x):
    return int(np.float32(x).view(np.uint32))


def unary(dm, what, x):
    xd = cu(x)
    y = torch.empty_like(xd)
    assert dm.dm_unary(what, ptr(xd), ptr(y), xd.numel()) == 0
    return y.cpu().numpy()


@pytest.mark.parametrize("what,lo,hi", [
    (RCP, 2.0 ** -40, 2.0 ** 60), (HALF_RSQRT, 2.0 ** -100, 2.0 ** 100)])
def test_every_float_of_the_range_has_the_operators_bits(dm, what, lo, hi):
    """The reciprocal for d in [2^-40, 2^60], 0.5 / sqrt(x) for x in [2^-100, 2^100]:
    all mantissas at all exponents, the all-ones one (the exception of a single Newton
    step from an estimate below 1/d) among them."""
    a, b = pattern(lo), pattern(hi)
    out = torch.tensor([0, -1], dtype=torch.int64, device="cuda")
    say(f"[sweep] form {what}: {b - a + 1} floats")
    while a <= b:
        n = min(b - a + 1, 1 << 28)
        assert dm.dm_sweep(what, C.c_uint32(a), C.c_uint32(n), ptr(out)) == 0
        a += n
    bad, first = out.cpu().numpy()
    say(f"[sweep] form {what}: {bad} differ, first {int(first) & 0xffffffffffffffff:#x}")
    assert bad == 0


@pytest.mark.parametrize("exponent", [-40, -8, 0, 1, 59])
def test_reciprocal_and_root_of_a_binade_against_numpy(dm, exponent):
    """the operators the ranges are compared with are IEEE's, and so are the short forms"""
    x = ((np.arange(1 << 23, dtype=np.uint32)) | np.uint32((exponent + 127) << 23)).view(np.float32)
    say(f"[binade] 2^{exponent}")
    one, half = np.float32(1), np.float32(0.5)
    for what, want in ((RCP, one / x), (HALF_RSQRT, half / np.sqrt(x))):
        np.testing.assert_array_equal(bits(unary(dm, what, x)), bits(want))
        np.testing.assert_array_equal(bits(unary(dm, what + OPERATORS, x)), bits(want))


def hard_quotients(rng, n):
    """(numerators, divisors): 24-bit significands N, D whose quotient lies r / (2^25 D)
    from a midpoint of two floats, r a small odd number of either sign: with
    D (2 Q + 1) = r modulo 2^25, N = (D (2 Q + 1) - r) / 2^25."""
    D = (rng.integers(1 << 23, 1 << 24, n) | 1).astype(np.int64)
    r = (2 * rng.integers(0, 8, n) + 1) * rng.choice([-1, 1], n)
    inv = D.copy()
    for _ in range(5):                       # the inverse modulo 2^25 (Newton)
        inv = inv * ((2 - D * inv) & 0x1ffffff) & 0x1ffffff
    m = inv * (r & 0x1ffffff) & 0x1ffffff    # 2 Q + 1
    N = (D * m - r) >> 25
    ok = (D * m - r == N << 25) & (N > 0)
    return N[ok], D[ok]


def test_quotients_next_to_midpoints(dm):
    """div_by against numpy's division: quotients a few 2^-49 from a rounding midpoint,
    exact ones, random ones, zeros of both signs, at the ends of the range it takes"""
    rng = np.random.default_rng(3)
    N, D = hard_quotients(rng, 1 << 22)
    assert len(N) > 1 << 21
    num = [N, rng.integers(1, 1 << 24, 1 << 22), rng.integers(1, 1 << 12, 1 << 20)]
    den = [D, rng.integers(1 << 23, 1 << 24, 1 << 22), rng.integers(1, 1 << 12, 1 << 20)]
    den[2], num[2] = den[2], num[2] * den[2]          # exact quotients
    ones = np.full(1 << 20, (1 << 24) - 1)
    num.append(rng.integers(1, 1 << 24, 1 << 20))     # by the all-ones significand
    den.append(ones)
    for a, d in zip(num, den):
        a, d = a.astype(np.float32), d.astype(np.float32)
        for ea, ed in ((0, 0), (-60, 60), (60, -40), (-60, -40), (60, 60), (3, -17)):
            # significands scaled into [2^ea, 2^(ea+1)), the numerator's top below 2^60
            sa = np.ldexp(np.frexp(a)[0], ea + (ea < 60)).astype(np.float32)
            sd = np.ldexp(np.frexp(d)[0], ed + (ed < 60)).astype(np.float32)
            sa[::3] *= -1
            sa[::1001] = 0.0
            sa[::1003] = -0.0
            say(f"[quotients] {len(sa)} at 2^{ea} / 2^{ed}")
            av, dv = cu(sa), cu(sd)
            q = torch.empty_like(av)
            assert dm.dm_div(ptr(av), ptr(dv), ptr(q), av.numel()) == 0
            np.testing.assert_array_equal(bits(q.cpu().numpy()), bits(sa / sd))


@pytest.mark.parametrize("share", [0.0, 0.002, 0.1, 0.9])
def test_projection_quotients_beside_lanes_out_of_range(dm, share):
    """hom_div with denominators at and below zero, zero, tiny, huge and non-finite
    numerators beside ordinary lanes of one wavefront (share of them; 0: none): the
    IEEE quotients where w > 0, position (0, 0) and false elsewhere"""
    rng = np.random.default_rng(int(share * 1000))
    n = 64 * 4096 + 37
    nu, nv = (rng.normal(size=n).astype(np.float32) * 2000 for _ in range(2))
    w = (1 + 0.2 * rng.normal(size=n)).astype(np.float32)
    w[w < 0.05] = 1.0
    odd = np.array([0.0, -0.0, 1e-30, 2.0 ** -60, 2.0 ** -61, 2.0 ** 60, 2.0 ** 61, 1e30, -1e30, np.inf, -np.inf, np.nan,
                    1e-40, -3.0], np.float32)
    for v in (nu, nv, w):
        k = rng.random(n) < share / 3
        v[k] = rng.choice(odd, k.sum())
    d = [cu(v) for v in (nu, nv, w)]
    u, v = torch.empty_like(d[0]), torch.empty_like(d[0])
    ok = torch.empty(n, dtype=torch.int32, device="cuda")
    say(f"[projection] share {share}")
    assert dm.dm_hom_div(*(ptr(t) for t in d), ptr(u), ptr(v), ptr(ok), n) == 0
    want = w > 0
    np.testing.assert_array_equal(ok.cpu().numpy() != 0, want)
    with np.errstate(all="ignore"):
        for got, num in ((u, nu), (v, nv)):
            q = np.where(want, num / w, np.float32(0))
            g = got.cpu().numpy()
            np.testing.assert_array_equal(np.isnan(g), np.isnan(q))
            np.testing.assert_array_equal(bits(g)[~np.isnan(q)], bits(q)[~np.isnan(q)])
