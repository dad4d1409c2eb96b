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
