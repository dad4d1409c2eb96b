"""Shifts of z-eigenbasis cube plans: those of a slice follow from its eigenvalue mu of A~, which
has to be known to full relative precision although the spectrum spans 30 n^4.  Reference:
Sturm-sequence bisection in extended precision.  Bound: mu to an ulp, and shifts that depend on
it smoothly, a few ulps, 1e-14."""
import numpy as np
import pytest

import paper_1710_11259_amd as fps

LD = np.longdouble


def eigenvalues(n, s):
    """Of -A~'s parity-s block, ascending, in extended precision."""
    j = np.arange(s, n, 2).astype(LD)
    d = 2 / ((2 * j + 1) * (2 * j + 5))
    e2 = 1 / ((2 * j + 5) ** 2 * (2 * j + 3) * (2 * j + 7))
    k = np.arange(len(j))
    lo, hi = np.full(len(j), LD(0.5) / (30 * LD(n) ** 4)), np.full(len(j), LD(1.01))
    for _ in range(100):
        x = np.where(hi > 2 * lo, np.sqrt(lo * hi), (lo + hi) / 2)
        q = d[0] - x
        below = (q < 0).astype(int)
        for i in range(1, len(j)):
            q = (d[i] - x) - e2[i - 1] / np.where(q == 0, LD(1e-300), q)
            below += q < 0
        lo, hi = np.where(below <= k, x, lo), np.where(below <= k, hi, x)
    return (lo + hi) / 2


@pytest.mark.parametrize("n", [3, 16, 64, 129])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refined"])
def test_longest_slice(n, precision):
    p = fps.plan(n, tol=1e-13, dim=3, zeig=True, precision=precision, host_only=True)
    got = np.array(p.shifts())
    tol = p.round_steps()[1][0] if precision != "fp64" else 1e-13
    b = 1.0 / (30.0 * n**4)
    best = np.inf
    for mu in np.concatenate([eigenvalues(n, 0), eigenvalues(n, 1)]).astype(float):
        if precision == "fp64":
            want = fps.adi_shifts(mu * mu / (1 + mu), mu * mu / (b + mu), b + mu, 1 + mu, tol)[0]
        else:
            lo, hi = mu + 0.5, mu / b + 0.5
            want = fps.adi_shifts(-hi, -lo, lo, hi, tol)[0][::-1]
        if len(want) == len(got):
            best = min(best, float(np.abs(np.array(want) / got - 1).max()))
    assert best <= 1e-14
