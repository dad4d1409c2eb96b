"""Rounding of the solves themselves: adjoints against a reference in extended precision,
cylinders by superposition.

On data that decay, what the truncation (tol = 1e-17 here) and the data leave is the
rounding of the products themselves.  Bound: the maps are rounded once per entry and
the partial sums of a product stay near its result, which is at most 1.5 u for each of the
four products, 6 u = 6.7e-16 in all (relative Frobenius norm, rms over three
inputs).  Maps whose own formation leaves a few u per entry exceed it, and so do sums
over modes that start with the largest terms."""
import numpy as np
import pytest

from oracle import basis, square

torch = pytest.importorskip("torch")
import paper_1710_11259_amd as fps  # noqa: E402

LD = np.longdouble


def sylvester(G):
    """Y with A~ Y + Y A~ = G: the oracle's float64 solve, refined with residuals in extended precision."""
    n = G.shape[0]
    j = np.arange(n).astype(LD)
    d = -2 / ((2 * j + 1) * (2 * j + 5))
    e = (1 / ((2 * j + 5) * np.sqrt((2 * j + 3) * (2 * j + 7))))[:-2, None]

    def left(Y):
        Z = d[:, None] * Y
        Z[:-2] += e * Y[2:]
        Z[2:] += e * Y[:-2]
        return Z

    eig = square.atilde_eig(n)
    Y = np.zeros_like(G)
    for _ in range(6):
        R = G - left(Y) - left(Y.T).T
        Y = Y + square.solve_symmetric_sylvester(R.astype(np.float64), eig)
    return Y


def adjoint(Ubar, out):
    n = Ubar.shape[0] - (2 if out == "cheb" else 0)
    s = np.sqrt((np.arange(n).astype(LD) + 1) * (np.arange(n) + 2))
    Ri = basis.cheb_to_ct(n, LD) / s[:, None]
    Po = basis.recombined_to_cheb(n, LD) / s if out == "cheb" else np.diag(1 / s)
    return Ri.T @ sylvester(Po.T @ Ubar.astype(LD) @ Po) @ Ri


def decaying(rng, m):
    w = (1.0 + np.arange(m)) ** -2
    return rng.standard_normal((m, m)) * np.outer(w, w)


@pytest.mark.gpu
@pytest.mark.parametrize("n,out", [(n, out) for n in (64, 256, 515) for out in ("cheb", "native")])
def test_adjoint(n, out):
    p = fps.plan(n, tol=1e-17, tight=True, out=out)
    errs = []
    for seed in range(3):
        Ubar = decaying(np.random.default_rng(seed), p.out_shape()[0])
        got = fps.solve_adjoint(p, torch.from_numpy(Ubar).cuda()).cpu().numpy()
        want = adjoint(Ubar, out)
        errs.append(float(np.linalg.norm((got - want).astype(float)) / np.linalg.norm(want.astype(float))))
    print(f"n={n} {out} rel err {errs}", flush=True)
    assert np.sqrt(np.mean(np.square(errs))) <= 6 * 2.0 ** -53


# U(A + B) - U(A) - U(B) for inputs whose sum is exact: what is left is rounding.  The banded
# solves magnify the rounding of their right-hand sides some 20 times at these sizes: 20 u
# sqrt(3) for three solves, 3.8e-15; with the right-hand sides' sums started from their
# largest terms it is 1e-14.
@pytest.mark.gpu
@pytest.mark.parametrize("n", [64, 130])
def test_cylinder_superposition(n):
    nt = 32
    p = fps.plan_cylinder(n, nt)
    k = np.abs(np.arange(nt) - nt // 2)
    i = np.arange(n)
    w = (1.0 + i) ** -2
    weight = ((1.0 + k) ** -2)[:, None, None, None] * w[:, None] * w
    weight = weight * ((i % 2)[None, :] == (k % 2)[:, None])[:, None, :, None]
    errs = []
    for seed in range(8):
        rng = np.random.default_rng(seed)
        A, B = (torch.from_numpy((rng.standard_normal((nt, 2, n, n)) * weight).astype(np.float32)).cuda().double()
                for _ in range(2))
        UA = fps.solve(p, A)
        errs.append(float((fps.solve(p, A + B) - UA - fps.solve(p, B)).norm() / UA.norm()))
    print(f"n={n} superposition {errs}", flush=True)
    assert np.sqrt(np.mean(np.square(errs))) <= 5e-15
