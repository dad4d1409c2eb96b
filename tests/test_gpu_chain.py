"""Chains of products on one LDS-resident block, at the sizes where their
tiles end: blocks of 32, 64, 96 and 128 entries and one off, the output rows
and columns past a whole block (up to 2), and the sizes on either side of
which the per-axis products take over (squares 128, cubes and cylinders
256).  Products of length n/2 round by a few hundred eps of the data: 1e-12."""
import numpy as np
import pytest

import parity
import workloads
from oracle import adjoint, cube, cylinder, square

torch = pytest.importorskip("torch")
import paper_1710_11259_amd as fps  # noqa: E402

pytestmark = pytest.mark.gpu


def _host(U):
    torch.cuda.synchronize()
    return U.cpu().numpy()


@pytest.mark.parametrize("n", [1, 31, 63, 64, 65, 95, 97, 126, 127, 128, 129, 130])
def test_square(n):
    rng = np.random.default_rng(n)
    F = rng.standard_normal((n, n))
    p = fps.plan(n, tol=1e-13)
    U = _host(fps.solve(p, torch.from_numpy(F).cuda()))
    parity.check(U, square.poisson_square(F), 1e-12, f"solve n={n}")
    Ub = rng.standard_normal(p.out_shape())
    Fb = _host(fps.solve_adjoint(p, torch.from_numpy(Ub).cuda()))
    parity.check(Fb, adjoint.vjp_square(Ub), 1e-12, f"adjoint n={n}")


def test_batch_of_chains_and_products():
    # chains of two block sizes and products in one batch, bitwise the single solves
    sizes = [128, 1, 300, 64, 127, 129, 2]
    rng = np.random.default_rng(0)
    Fs = [torch.from_numpy(rng.standard_normal((n, n))).cuda() for n in sizes]
    b = fps.batch(sizes, tol=1e-13)
    Us = b.unpack(fps.batch_solve(b, b.pack(Fs)))
    for n, F, U in zip(sizes, Fs, Us):
        assert torch.equal(U, fps.solve(fps.plan(n, tol=1e-13), F)), n


@pytest.mark.parametrize("n", [31, 65, 127, 130, 191, 193, 254, 255, 257])
@pytest.mark.parametrize("out", ["cheb", "native"])
def test_cube(n, out):
    F = workloads.cube_rhs(n)
    p = fps.plan(n, tol=1e-13, dim=3, out=out, zeig=True)
    U = _host(fps.solve(p, torch.from_numpy(F).cuda()))
    parity.check(U, cube.poisson_cube(F, out=out), 1e-12, f"cube n={n} {out}")


@pytest.mark.parametrize("n", [62, 66, 126, 128, 130, 190, 192, 194, 252, 256])
def test_cylinder(n):
    F = workloads.cylinder_rhs(n, 6, seed=n)
    x = torch.from_numpy(np.ascontiguousarray(np.stack([F.real, F.imag], axis=1))).cuda()
    p = fps.plan_cylinder(n, 6)
    # every entry of U is written: the rows of the other parity are zero
    U = torch.full(p.out_shape(), float("nan"), dtype=torch.float64, device="cuda")
    u = _host(fps.solve(p, x, out=U))
    parity.check(u[:, 0] + 1j * u[:, 1], cylinder.poisson_cylinder(F), 1e-12, f"cylinder n={n}")
