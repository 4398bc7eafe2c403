"""CPU check of the floating-point transforms' bounds (csrc/ntt_field.hpp): the
butterflies level by level in IEEE doubles with the reductions where the
kernels place them, for the largest primes of both classes and inputs at the
ends of the range.  Every intermediate value must stay below 2^53 in absolute
value (so that each operation is exact) and the inverse must give back n times
the input."""
import numpy as np
import pytest

from oracle import bfv

LIM = 2.0 ** 53


def mulmod(y, w, wi, p):
    """y w - rint(y w/p) p with the kernel's rounding of the quotient; exact."""
    assert np.abs(y).max() < LIM
    g = np.rint(y * wi)
    ints = [np.array([int(v) for v in a], dtype=object) for a in (y, w, g)]
    out = (ints[0] * ints[1] - ints[2] * p).astype(np.float64)
    assert (np.abs(out) < LIM).all()
    return out


def red(x, p):
    assert np.abs(x).max() <= LIM
    g = np.rint(x * (1.0 / p))
    return np.array([int(v) - int(q) * p for v, q in zip(x, g)], dtype=object).astype(np.float64)  # one fma, exact


def passes(L):
    full = [(P, 4, L - 4 * P - 4) for P in range(L // 4)]
    return full + ([(L // 4, L % 4, 0)] if L % 4 else [])


def transform(x, tw, p, L, inverse, big):
    n = 1 << L
    idx = np.arange(n)
    ps = passes(L)
    for P, r, lo in (ps[::-1] if inverse else ps):
        if big and not inverse and P in (1, 3):  # entry of the block part, before its third pass
            x = red(x, p)
        for u in (range(r - 1, -1, -1) if inverse else range(r)):
            lev = 4 * P + u
            half = n >> (lev + 1)
            X, Y = idx[(idx & half) == 0], idx[(idx & half) != 0]
            W = tw[(1 << lev) + (X >> (L - lev))]
            wi = W / p
            if inverse and big and r == 4 and u == 0:
                s = (idx >> lo) & 15
                sel = (s & 7) <= 1
                x[sel] = red(x[sel], p)
            a, b = x[X].copy(), x[Y].copy()
            if inverse:
                x[X] = a + b
                x[Y] = mulmod(a - b, W, wi, p)
            else:
                t = mulmod(b, W, wi, p)
                x[X], x[Y] = a + t, a - t
            assert np.abs(x).max() < LIM
        if inverse:
            s = (idx >> lo) & ((1 << r) - 1)
            sel = s < ((8 if big else 4) if r == 4 else (1 << r) // 2)
            x[sel] = red(x[sel], p)
    return x


@pytest.mark.parametrize("L", [12, 13, 14])
@pytest.mark.parametrize("bits", [47, 50])
def test_bounds_and_round_trip(L, bits):
    n = 1 << L
    p = bfv.ntt_primes(n, bits, 1)[0]
    big = p >= 1 << 47
    psi = next(c for c in (pow(x, (p - 1) // (2 * n), p) for x in range(2, 200)) if pow(c, n, p) == p - 1)
    rev = [int(format(i, f"0{L}b")[::-1], 2) for i in range(n)]
    pw = [1] * n
    for i in range(1, n):
        pw[i] = pw[i - 1] * psi % p
    ipsi = pow(psi, -1, p)
    ipw = [1] * n
    for i in range(1, n):
        ipw[i] = ipw[i - 1] * ipsi % p
    centre = lambda v: float(v - p if v > p // 2 else v)  # noqa: E731
    tw = np.array([centre(pw[r]) for r in rev])
    itw = np.array([centre(ipw[r]) for r in rev])
    rng = np.random.default_rng(L * bits)
    for src in (np.full(n, p - 1, dtype=np.int64), np.where(np.arange(n) % 2, p - 1, 0), rng.integers(0, p, n)):
        y = transform(src.astype(np.float64), tw, p, L, False, big)
        # products enter the inverse below 0.51 p (reduced sums)
        z = transform(red(y, p), itw, p, L, True, big)
        assert np.abs(z).max() < 2.1 * p  # a constant multiple of it is then below p in absolute value
        for i in list(range(8)) + [n // 2, n - 1]:
            assert int(z[i]) % p == int(src[i]) * n % p
