"""The reciprocal-based quotient and the square root of the hot loops at the
edges of their fast forms: signed zeros, powers of two, divisors with every
mantissa bit (or the whole low word) set, and operands on both sides of the
range limits 2^+-400 and 2^+-600.  The host's IEEE-754 results are the
reference, bit for bit (the sign of a zero included)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _edges():
    one = np.float64(1.0)
    mant = [one, np.nextafter(one, 2), np.nextafter(np.float64(2), 1), np.float64(1.5),
            np.float64((2 ** 52 + 0xffffffff) / 2 ** 52), np.float64(4 / 3)]
    b = [np.ldexp(m, e) for m in mant for e in (-401, -400, -399, -1, 0, 1, 398, 399, 400)]
    a = [np.ldexp(m, e) for m in mant for e in (-601, -600, -599, -3, 0, 5, 598, 599, 600)]
    a = np.array(a + [0.0])
    a = np.concatenate([a, -a])
    A, Bm = np.meshgrid(a, np.array(b), indexing="ij")
    A, Bm = A.ravel(), Bm.ravel()
    with np.errstate(all="ignore"):
        q = np.abs(A / Bm)
    keep = (A == 0.0) | ((q >= 2.0 ** -900) & (q <= 2.0 ** 900))
    return A[keep], Bm[keep]


@pytest.mark.parametrize("seed", [0, 1])
def test_quotient_edges(seed):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_09145_amd import binding as B
    a, b = _edges()
    # random dividends against the edge divisors, and divisors whose low word is all ones
    rng = np.random.default_rng(seed)
    ra = rng.standard_normal(200_000) * 2.0 ** rng.integers(-200, 200, 200_000)
    rb = np.abs(rng.standard_normal(200_000)) + 1e-3
    rb = (rb.view(np.uint64) | np.uint64(0xffffffff)).view(np.float64)
    a = np.concatenate([a, ra, ra])
    b = np.concatenate([b, rb, rng.choice(_edges()[1], 200_000)])
    with np.errstate(all="ignore"):
        keep = (a == 0.0) | ((np.abs(a / b) >= 2.0 ** -900) & (np.abs(a / b) <= 2.0 ** 900))
    a, b = a[keep], b[keep]
    ad, bd = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    _, q2, _, _ = B.selftest_arith(ad, bd)
    _, _, s, _ = B.selftest_arith(bd, bd)
    torch.cuda.synchronize()
    assert np.array_equal(q2.cpu().numpy().view(np.int64), (a / b).view(np.int64))
    assert np.array_equal(s.cpu().numpy().view(np.int64), np.sqrt(b).view(np.int64))
