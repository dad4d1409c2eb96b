"""The eigenbasis form of the 2-D solves: four products with the shifts'
error factors in between must give the J-step iterate of Algorithm 2, not
just any solution within tol, so loose tolerances are compared with the
oracle's closed form of that iterate.  Bound: the truncation is common to
both sides, so only rounding differs (products of length n/2 and the factors
of up to 60 steps, a few hundred eps): 1e-12."""
import numpy as np
import pytest

import parity
from oracle import basis, rect, square

torch = pytest.importorskip("torch")
import paper_1710_11259_amd as fps  # noqa: E402

pytestmark = pytest.mark.gpu

BOX = (0.0, 2.5, -1.0, 0.25)


def _run(p, F):
    U = fps.solve(p, torch.from_numpy(np.ascontiguousarray(F)).cuda())
    torch.cuda.synchronize()
    return U.cpu().numpy()


# sizes around the parity padding (64) and the product tiles (128), the
# smallest ones, and one of several tiles
@pytest.mark.parametrize("n", [1, 2, 3, 126, 127, 128, 129, 255, 258, 513])
@pytest.mark.parametrize("tol", [0.3, 1e-4])
def test_square_is_the_j_step_iterate(n, tol):
    F = np.random.default_rng(n).standard_normal((n, n))
    p = fps.plan(n, tol=tol)
    parity.check(_run(p, F), square.poisson_square_adi(F, np.array(p.shifts())), 1e-12, f"n={n}")
    q = fps.plan(n, tol=tol, out="native", tight=True)
    want = square.poisson_square_adi(F, np.array(q.shifts()), out="native")
    parity.check(_run(q, F), want, 1e-12, f"native n={n}")


@pytest.mark.parametrize("n", [2, 65, 300])
def test_rect_is_the_j_step_iterate(n):
    F = np.random.default_rng(n).standard_normal((n, n))
    p = fps.plan(n, tol=1e-3, box=BOX)
    sp, sq = (np.array(v) for v in p.shift_pairs())
    s = square.s_diag(n)
    Y = rect.adi_iterate_rect(square.rhs_ct(F) / np.outer(s, s), BOX, sp, sq)
    P = basis.recombined_to_cheb(n)
    parity.check(_run(p, F), P @ (Y / np.outer(s, s)) @ P.T, 1e-12, f"rect n={n}")


def test_adjoint_of_a_loose_solve():
    # <U(F), Ubar> = <F, Fbar> for the same J-step map
    n = 131
    rng = np.random.default_rng(7)
    for out in ("cheb", "native"):
        p = fps.plan(n, tol=1e-2, out=out, box=BOX)
        F, Ub = rng.standard_normal((n, n)), rng.standard_normal(p.out_shape())
        U = _run(p, F)
        Fb = fps.solve_adjoint(p, torch.from_numpy(Ub).cuda()).cpu().numpy()
        a, b = (U * Ub).sum(), (F * Fb).sum()
        scale = np.linalg.norm(U) * np.linalg.norm(Ub)
        assert abs(a - b) <= 1e-13 * scale


# Sizes at which the output map's zeros (modes below a row's limit) are skipped,
# by both tiles, with edge rows (n = 1025: 513 and 513 coefficients) and without;
# undecayed data, so that every coefficient weighs the same.
@pytest.mark.parametrize("n,out", [(300, "cheb"), (700, "native"), (1025, "cheb"), (1800, "cheb")])
def test_skipped_zeros_of_the_output_map(n, out):
    from oracle import adjoint
    rng = np.random.default_rng(n)
    p = fps.plan(n, tol=1e-13, out=out, tight=True)
    F = rng.standard_normal((n, n))
    parity.check(_run(p, F), square.poisson_square(F, out=out), 1e-12, f"solve n={n}")
    if out == "cheb":
        Ub = rng.standard_normal(p.out_shape())
        Fb = fps.solve_adjoint(p, torch.from_numpy(Ub).cuda()).cpu().numpy()
        parity.check(Fb, adjoint.vjp_square(Ub), 1e-12, f"adjoint n={n}")


# The cube's multiplier against the iterations written out with dense solves.
# Their matrices K = -A~^-1 have condition 30 n^4, so the oracle carries
# 30 n^4 eps (1.4e-11 at n = 8) and the bound is 1e-9; the truncation being
# compared is about 1e-2.
@pytest.mark.parametrize("n", [3, 8])
@pytest.mark.parametrize("method", ["nested", "zeig", "refined"])
def test_cube_is_the_iterate_of_its_method(n, method):
    from oracle import cube
    tol = 1e-2
    F = np.random.default_rng(n).standard_normal((n, n, n))
    G = cube.symmetric_rhs(cube.rhs_ct(F))
    p = fps.plan(n, tol=tol, dim=3, out="native", tight=method == "zeig", zeig=method != "nested",
                 precision="fp32_refined" if method == "refined" else "fp64")
    s = square.s_diag(n)
    X = _run(p, F) * s[:, None, None] * s[None, :, None] * s[None, None, :]
    if method == "nested":
        Y, J, inner = cube.kform_adi(G, tol, 0.1 * tol)
        assert J == p.J and inner == p.inner_counts()
    elif method == "zeig":
        Y, counts = cube.zeig_adi(G, tol)
        assert sorted(counts, reverse=True) == p.slice_counts()
    else:
        # one round: symmetric shifts on [|mu| / |lmin| + 1/2, |mu| / |lmax| + 1/2]
        steps, tols = p.round_steps()
        assert len(steps) == 1
        lam, V = square.atilde_eig(n)
        Gh = G
        for m in range(3):
            Gh = cube.mode_product(Gh, V.T, m)
        Yh = np.empty_like(Gh)
        for c, mu in enumerate(lam):
            a, b = abs(mu) + 0.5, abs(mu) * 30.0 * n ** 4 + 0.5
            ps, qs = fps.adi_shifts(-b, -a, a, b, tols[0])
            z = -(abs(mu) * (-1.0 / lam) + 0.5)
            r = np.prod([(z - pj) / (z - qj) for pj, qj in zip(ps, qs)], axis=0)
            den = lam[:, None] * lam[None, :] + mu * (lam[:, None] + lam[None, :])
            Yh[c] = -Gh[c] * (1.0 - np.outer(r, r)) / den
        Y = Yh
        for m in range(3):
            Y = cube.mode_product(Y, V, m)
    parity.check(X, Y, 1e-9, f"cube {method} n={n}")
