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


# Inputs read in natural order by the first product: odd sizes (the last column
# stands alone), odd offsets (rows 8-byte aligned only), sizes around the tiles, and
# values beyond the array that must not matter.
@pytest.mark.parametrize("n", [129, 130, 191, 257, 515, 1023, 1026])
@pytest.mark.parametrize("offset", [0, 1])
def test_natural_input(n, offset):
    rng = np.random.default_rng(n)
    p = fps.plan(n, tol=1e-13)

    def padded(x):
        buf = torch.full((x.size + 64,), float("nan"), dtype=torch.float64, device="cuda")
        v = buf[offset:offset + x.size].view(x.shape)
        v.copy_(torch.from_numpy(x))
        return v

    F = rng.standard_normal((n, n))
    parity.check(_host(fps.solve(p, padded(F))), square.poisson_square(F), 1e-12, f"solve n={n}")
    Ub = rng.standard_normal(p.out_shape())
    parity.check(_host(fps.solve_adjoint(p, padded(Ub))), adjoint.vjp_square(Ub), 1e-12, f"adjoint n={n}")


# F and U may overlap in any way: every input is read before an output is written.
@pytest.mark.parametrize("ns", [[1], [1, 2, 1], [40, 128], [33, 200, 1]])
@pytest.mark.parametrize("out", ["cheb", "native"])
@pytest.mark.parametrize("shift", [0, 3])
def test_overlapping_input_and_output(ns, out, shift):
    rng = np.random.default_rng(len(ns))
    b = fps.batch(ns, tol=1e-13, out=out)
    F = torch.from_numpy(rng.standard_normal(b.in_entries)).cuda()
    U = fps.batch_solve(b, F)
    buf = torch.zeros(b.out_entries + 8, dtype=torch.float64, device="cuda")
    x = buf[shift:shift + b.in_entries]
    x.copy_(F)
    y = fps.batch_solve(b, x, out=buf[:b.out_entries])
    parity.check(_host(y), U.cpu().numpy(), 1e-13, "batch")
    n = ns[0]
    p = fps.plan(n, tol=1e-13, out=out)
    F1 = F[:n * n].view(n, n)
    U1 = fps.solve(p, F1)
    x = buf[shift:shift + n * n].view(n, n)
    x.copy_(F1)
    y = fps.solve(p, x, out=buf[:U1.numel()].view(U1.shape))
    parity.check(_host(y), U1.cpu().numpy(), 1e-13, "single")


# Banded solves with and without row exchanges: only the systems of |k| = 2 have
# them, from n = 130 on in some of the 64-column blocks alone.  Per mode, so that no
# mode hides behind a larger one.
@pytest.mark.parametrize("n", [2, 4, 16, 64, 130, 256, 300])
def test_cylinder_modes_with_row_exchanges(n):
    F = workloads.cylinder_rhs(n, 6, seed=n + 1)
    x = torch.from_numpy(np.ascontiguousarray(np.stack([F.real, F.imag], axis=1))).cuda()
    u = _host(fps.solve(fps.plan_cylinder(n, 6), x))
    for k in (-2, 2, -3, 1):
        Fk = F[k + 3]
        Uk = (cylinder.solve_mode(np.ascontiguousarray(Fk.real), k)
              + 1j * cylinder.solve_mode(np.ascontiguousarray(Fk.imag), k))
        parity.check(u[k + 3, 0] + 1j * u[k + 3, 1], Uk, 1e-12, f"cylinder n={n} mode {k}")


# Banded solves on both sides of 512 units, from which the halves of a |k| group share
# a workgroup: 3 blocks of columns, the last one partly past the padded size, times
# 170 and 171 groups, of which k = 0 and -n_theta / 2 have one half alone.
@pytest.mark.parametrize("nt", [338, 340])
def test_cylinder_many_modes(nt):
    n = 130
    F = workloads.cylinder_rhs(n, nt, seed=nt)
    x = torch.from_numpy(np.ascontiguousarray(np.stack([F.real, F.imag], axis=1))).cuda()
    u = _host(fps.solve(fps.plan_cylinder(n, nt), x))
    for k in (0, -1, 2, -2, 57, nt // 2 - 1, -(nt // 2)):
        Fk = F[k + nt // 2]
        Uk = (cylinder.solve_mode(np.ascontiguousarray(Fk.real), k)
              + 1j * cylinder.solve_mode(np.ascontiguousarray(Fk.imag), k))
        parity.check(u[k + nt // 2, 0] + 1j * u[k + nt // 2, 1], Uk, 1e-12, f"mode {k}")
