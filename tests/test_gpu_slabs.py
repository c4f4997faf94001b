"""Launches in slab order (lattices without whole-tile z-groups) at every
site: the fused operator against the operator composed of whole-lattice
shifts, colour products and projectors, which share no traversal with it, and
the block sums of a solve through the residual of its result."""

import pytest
import torch

import lattice_inputs as LI
import paper_2001_07557_amd as P

pytestmark = pytest.mark.gpu

# 162-site planes and a ragged last tile; 392-site planes; six and ten planes
# (both-parity launches only), the last slab of a slice short of its pad
DIMS = [(18, 18, 42, 40), (28, 28, 28, 28), (46, 46, 6, 60), (30, 30, 10, 60)]
# 24 launches of rounded intermediates against FMA chains, per site against its
# largest entry: a hundred units of the working precision
TOL = {P.F64: 100 * 1.1e-16, P.F32: 100 * 6e-8}


def close(a, b, tol):
    d = (a - b).abs().amax((-1, -2))
    return bool((d <= tol * b.abs().amax((-1, -2))).all())


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec,link", [(P.F64, 18), (P.F64, 12), (P.F32, 18), (P.F32, 12)])
def test_every_site_against_generic(dims, prec, link):
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields_device(9, dims, "cuda")
    Uf, x = P.pack_gauge(lat, U, prec, link), P.pack_spinor(lat, psi, prec)
    out, t1, t2 = (P.new_spinor(lat, prec, P.FULL) for _ in range(3))
    for dagger in (False, True):
        want = P.unpack_spinor(P.dslash_generic(out, x, Uf, t1, t2, dagger=dagger))
        out.buf.zero_()
        assert close(P.unpack_spinor(P.dslash(out, x, Uf, dagger=dagger)), want, TOL[prec])
        out.buf.zero_()
        P.meo(out.half(P.EVEN), x.half(P.ODD), Uf, dagger=dagger)
        P.moe(out.half(P.ODD), x.half(P.EVEN), Uf, dagger=dagger)
        assert close(P.unpack_spinor(out), want, TOL[prec])


@pytest.mark.parametrize("prec,link", [(P.F64, 18), (P.F32, 12), (P.F16, 12)])
def test_solve_in_slab_order(prec, link):
    dims, kappa, tol = (18, 18, 42, 40), 0.12, 1e-10
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields_device(10, dims, "cuda")
    hi = P.pack_gauge(lat, U, P.F64, 18)
    lo = hi if prec == P.F64 else P.pack_gauge(lat, U, prec, link)
    b = P.pack_spinor(lat, psi, P.F64, P.EVEN)
    x, mx, ax = (P.new_spinor(lat, P.F64, P.EVEN) for _ in range(3))
    tmp = P.new_spinor(lat, P.F64, P.ODD)
    st = P.cg_solve(x, b, hi, lo, kappa, tol=tol)
    P.mhat(mx, x, tmp, hi, kappa)
    P.mhat(ax, mx, tmp, hi, kappa, dagger=True)
    bb = P.norm2(b)
    P.axpby(1.0, b, -1.0, ax)
    res = (P.norm2(ax) / bb) ** 0.5
    assert res <= tol and abs(res - st.true_residual) <= 1e-3 * tol
