"""A solve whose last tile has fewer sites (8) than the lattice has block sums
(11), so that a sum formed by the active lanes of that tile alone would miss
some, and one that takes hundreds of iterations."""

import pytest

import lattice_inputs as LI
import paper_2001_07557_amd as P

pytestmark = pytest.mark.gpu


def solve(dims, kappa, tol, prec, seed=51):
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields_device(seed, dims, "cuda")
    hi = P.pack_gauge(lat, U, P.F64, 12)
    lo = hi if prec == P.F64 else P.pack_gauge(lat, U, prec, 12)
    b = P.pack_spinor(lat, psi, P.F64, P.EVEN)
    x, mx, ax = (P.new_spinor(lat, P.F64, P.EVEN) for _ in range(3))
    tmp = P.new_spinor(lat, P.F64, P.ODD)
    st = P.cg_solve(x, b, hi, lo, kappa, tol=tol)
    P.mhat(mx, x, tmp, hi, kappa)
    P.mhat(ax, mx, tmp, hi, kappa, dagger=True)
    bb = P.norm2(b)
    P.axpby(1.0, b, -1.0, ax)
    assert (P.norm2(ax) / bb) ** 0.5 <= tol
    return st.iterations


@pytest.mark.parametrize("prec", [P.F64, P.F32, P.F16])
def test_fewer_sites_in_the_last_tile_than_sums(prec):
    dims = (2, 6, 6, 18)
    ref = solve(dims, 0.12, 1e-10, P.F64)
    n = solve(dims, 0.12, 1e-10, prec)
    assert n <= ref * (1.0 if prec == P.F64 else 1.1 if prec == P.F32 else 1.6) + 2


@pytest.mark.parametrize("tol", [1e-10, 1e-12])
def test_fp32_iterations_on_an_ill_conditioned_system(tol):
    """The FP32 recurrence may drift four decades, or six where an update is
    put off, between updates; what that costs in iterations stays within a
    tenth, and ten between two reads."""
    dims, kappa = (8, 8, 8, 8), 0.22
    ref = solve(dims, kappa, tol, P.F64)
    assert ref > 200
    assert solve(dims, kappa, tol, P.F32) <= 1.1 * ref + 10
