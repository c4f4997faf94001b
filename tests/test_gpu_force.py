"""GPU parity of the fermion-force kernel and the autograd wrapper.

Raw link gradients and su(3) forces are compared with the FP64 oracle
(FP64 <= 1e-13, FP32 <= 2e-6 relative); the autograd function is checked
with torch.autograd.gradcheck on 2^4 and, on the 24^4 workload, with
central finite differences (h = 1e-6, FP64) of S = |M psi|^2 on 64 random
site entries and 64 random link entries, through the same 12-real forward
that is differentiated.  The finite differences sum
|phi(y)|^2 only over the sites a perturbation can change, which is the same
difference of S without the cancellation of the full-lattice sum.
"""

import numpy as np
import pytest
import torch

import lattice_inputs as LI
import paper_2001_07557_amd as P
from oracle import dirac, force, links, solver
from tests.gpu_helpers import dev, f32, host, rel, site_rel

pytestmark = pytest.mark.gpu

KAPPA = 0.124


@pytest.mark.parametrize("dims,bc", [((4, 4, 4, 4), (1, 1, 1, -1)), ((6, 4, 2, 6), (-1, 1, 1, -1)),
                                     ((2, 2, 2, 2), (1, 1, 1, -1))])
@pytest.mark.parametrize("prec,link", [(P.F64, 18), (P.F64, 12), (P.F32, 18), (P.F32, 12)])
def test_force_kernel_vs_oracle(dims, bc, prec, link):
    lat = P.Lattice(dims, bc)
    U, X = LI.workload_fields(30, dims)
    Y = LI.gaussian_spinor(np.random.default_rng(31), dims)
    c0 = -0.37
    if prec == P.F32:
        Ur, Xr, Yr, tdt, tol = f32(U), f32(X), f32(Y), torch.complex64, 2e-6
        if link == 12:
            Ur = links.reconstruct(links.compress(Ur))
    else:
        Ur, Xr, Yr, tdt, tol = U, X, Y, torch.complex128, 1e-13
    Uf = P.pack_gauge(lat, dev(U).to(tdt), prec, link)
    Xf = P.pack_spinor(lat, dev(X).to(tdt), prec)
    Yf = P.pack_spinor(lat, dev(Y).to(tdt), prec)
    G = force.link_gradient(Xr, Yr, Ur, c0, bc)
    F = force.su3_force(G, Ur)
    got_g = host(P.unpack_gauge(P.fermion_force(Xf, Yf, Uf, c0, mode=1)))
    assert rel(got_g, G) < tol
    assert site_rel(got_g, G, per=9) < tol
    out = P.fermion_force(Xf, Yf, Uf, c0, mode=0)
    got_f = host(P.unpack_gauge(out))
    assert rel(got_f, F) < tol
    assert site_rel(got_f, F, per=9) < tol
    # accumulate adds to the existing field
    P.fermion_force(Xf, Yf, Uf, c0, mode=0, out=out, accumulate=True)
    assert rel(host(P.unpack_gauge(out)), 2 * F) < tol
    if link == 12:
        # the gradient carried onto the stored rows 0 and 1 (row 2 zero)
        rows = Ur if prec == P.F64 else f32(U)
        want = force.rows01_gradient(G, rows)
        got = host(P.unpack_gauge(P.fermion_force(Xf, Yf, Uf, c0, mode=2)))
        assert rel(got, want) < tol
        assert site_rel(got, want, per=9) < tol


@pytest.mark.parametrize("link", [P.LINK18, P.LINK12])
def test_autograd_gradcheck_2x4(link):
    """gradcheck perturbs every real entry of U: with 12-real links the
    operator reads rows 0 and 1 only and rebuilds row 2, so the gradient
    with respect to the stored row 2 is zero and rows 0, 1 carry the chain
    through the rebuild."""
    dims = (2, 2, 2, 2)
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields(32, dims)
    tpsi = dev(psi).requires_grad_(True)
    tU = dev(U).requires_grad_(True)
    f = lambda a, b: P.wilson_matrix(a, b, KAPPA, lat, P.F64, link)  # noqa: E731
    assert torch.autograd.gradcheck(f, (tpsi, tU), eps=1e-6, atol=1e-8, rtol=1e-7)


@pytest.mark.parametrize("prec,link", [(P.F64, 18), (P.F64, 12), (P.F32, 12)])
def test_autograd_vjp_vs_oracle(prec, link):
    dims = (8, 4, 6, 4)
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields(33, dims)
    g = LI.gaussian_spinor(np.random.default_rng(34), dims)
    tdt = torch.complex64 if prec == P.F32 else torch.complex128
    tpsi = dev(psi).to(tdt).requires_grad_(True)
    tU = dev(U).to(tdt).requires_grad_(True)
    phi = P.wilson_matrix(tpsi, tU, KAPPA, lat, prec, link)
    phi.backward(dev(g).to(tdt))
    want_phi = dirac.wilson(psi, U, KAPPA)
    want_gpsi, want_gU = force.vjp(psi, U, KAPPA, g)
    if link == 12:
        want_gU = force.rows01_gradient(want_gU, U)
    tol = 2e-6 if prec == P.F32 else 1e-13
    assert rel(host(phi).astype(np.complex128), want_phi) < tol
    assert rel(host(tpsi.grad).astype(np.complex128), want_gpsi) < tol
    assert rel(host(tU.grad).astype(np.complex128), want_gU) < tol
    if prec == P.F32:
        assert site_rel(host(phi), want_phi) < tol
        assert site_rel(host(tpsi.grad), want_gpsi) < tol
        assert site_rel(host(tU.grad), want_gU, per=9) < tol


def test_autograd_su3_force_mode():
    dims = (4, 4, 4, 4)
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields(35, dims)
    tpsi = dev(psi).requires_grad_(True)
    tU = dev(U).requires_grad_(True)
    phi = P.wilson_matrix(tpsi, tU, KAPPA, lat, P.F64, P.LINK12, link_grad="su3")
    (phi.abs() ** 2).sum().backward()
    want = force.su3_force(force.grad_links_norm(psi, U, KAPPA), U)
    assert rel(host(tU.grad), want) < 1e-13


# ----------------------------------------------------------------------------
# the 24^4 differentiated workload
# ----------------------------------------------------------------------------

def _touched_sites(dims, site):
    """Sites whose M psi depends on psi(site): the site and its 8 neighbours."""
    x, y, z, t = site
    out = {(x, y, z, t)}
    for mu in range(4):
        for s in (1, -1):
            c = [x, y, z, t]
            c[mu] = (c[mu] + s) % dims[mu]
            out.add(tuple(c))
    return sorted(out)


def _local_s(phi, sites):
    return sum(float(np.vdot(phi[t, z, y, x], phi[t, z, y, x]).real) for (x, y, z, t) in sites)


@pytest.mark.slow
@pytest.mark.parametrize("prec", [P.F64, P.F32])
def test_differentiated_24x4(prec):
    dims = (24, 24, 24, 24)
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields(3, dims)
    tdt = torch.complex64 if prec == P.F32 else torch.complex128
    tpsi = dev(psi).to(tdt).requires_grad_(True)
    tU = dev(U).to(tdt).requires_grad_(True)
    phi = P.wilson_matrix(tpsi, tU, KAPPA, lat, prec, P.LINK12)
    (phi.abs() ** 2).sum().backward()
    gpsi = host(tpsi.grad).astype(np.complex128)
    gU = host(tU.grad).astype(np.complex128)
    # against the oracle gradient (FP64 oracle on FP64 inputs for both
    # precisions; 12-real links: the gradient on the stored rows 0 and 1)
    want_gpsi = force.grad_psi_norm(psi, U, KAPPA)
    want_gU = force.rows01_gradient(force.grad_links_norm(psi, U, KAPPA), U)
    tol = 2e-6 if prec == P.F32 else 1e-13
    assert rel(gpsi, want_gpsi) < tol
    assert rel(gU, want_gU) < tol
    if prec != P.F64:
        assert site_rel(gpsi, want_gpsi) < tol
        assert site_rel(gU, want_gU, per=9) < tol
        return
    # central finite differences on the same GPU forward (12-real links),
    # h = 1e-6; entries of the stored row 2 have zero gradient
    rng = LI.fd_rng(4)
    h = 1e-6
    Ut = dev(U)

    def phi_of(ps, uu):
        with torch.no_grad():
            return host(P.wilson_matrix(ps, uu, KAPPA, lat, P.F64, P.LINK12))

    worst = 0.0
    for _ in range(64):
        site = tuple(int(rng.integers(0, d)) for d in dims)
        s, c = int(rng.integers(0, 4)), int(rng.integers(0, 3))
        part = 1.0 if rng.integers(0, 2) == 0 else 1j
        sites = _touched_sites(dims, site)
        idx = (site[3], site[2], site[1], site[0], s, c)
        pp = psi.copy(); pp[idx] += part * h
        pm = psi.copy(); pm[idx] -= part * h
        fd = (_local_s(phi_of(dev(pp), Ut), sites) - _local_s(phi_of(dev(pm), Ut), sites)) / (2 * h)
        an = gpsi[idx].real if part == 1.0 else gpsi[idx].imag
        worst = max(worst, abs(fd - an) / max(1.0, abs(an)))
    assert worst < 1e-6
    tp = dev(psi)
    worst = 0.0
    for _ in range(64):
        site = tuple(int(rng.integers(0, d)) for d in dims)
        mu, i, j = int(rng.integers(0, 4)), int(rng.integers(0, 3)), int(rng.integers(0, 3))
        part = 1.0 if rng.integers(0, 2) == 0 else 1j
        up = list(site)
        up[mu] = (up[mu] + 1) % dims[mu]
        sites = sorted({site, tuple(up)})
        idx = (site[3], site[2], site[1], site[0], mu, i, j)
        Up = U.copy(); Up[idx] += part * h
        Um = U.copy(); Um[idx] -= part * h
        fd = (_local_s(phi_of(tp, dev(Up)), sites) - _local_s(phi_of(tp, dev(Um)), sites)) / (2 * h)
        an = gU[idx].real if part == 1.0 else gU[idx].imag
        worst = max(worst, abs(fd - an) / max(1.0, abs(an)))
    assert worst < 1e-6


@pytest.mark.slow
def test_pseudofermion_force_pipeline_small():
    """Solve then force on the GPU (X_e from CG, X_o, Y_e, Y_o recomputed by
    hops) against the oracle's pseudofermion force from the same X_e."""
    dims = (8, 8, 8, 8)
    lat = P.Lattice(dims)
    U, phi = LI.workload_fields(36, dims)
    U_hi = P.pack_gauge(lat, dev(U), P.F64, 18)
    U_lo = P.pack_gauge(lat, dev(U).to(torch.complex64), P.F32, 12)
    b = P.pack_spinor(lat, dev(phi), P.F64, P.EVEN)
    F, st, x, _, _ = P.solve_and_force(b, U_hi, U_lo, KAPPA, tol=1e-12, U_force=U_hi)
    assert st.status == 0 and st.iterations < 200, st
    x_e = host(P.unpack_spinor(x))
    want = force.pseudofermion_force(x_e, U, KAPPA)
    assert rel(host(P.unpack_gauge(F)), want) < 1e-12
    assert solver.true_residual(x_e, dirac.project(phi, 0), U, KAPPA) <= 1.0001e-12


@pytest.mark.slow
def test_solve_and_force_48x3x96():
    """The 48^3x96 solve-plus-force workload: FP32 12-real smoothed links
    (kappa 0.1245), mixed CG to 1e-10, recomputed X_o, Y_e, Y_o, FP32 force.
    The residual is recomputed in FP64 through the operator entry points,
    the recomputed X_o, Y_e, Y_o are checked stage by stage against the
    oracle's hop of the previous stage, and the force against the oracle's
    link formula at 128 sampled links (FP64 arithmetic on the same stored
    X, Y and links)."""
    from tests.gpu_helpers import DeviceGather
    dims = (48, 48, 48, 96)
    kappa = 0.1245
    lat = P.Lattice(dims)
    Ud, psid = LI.workload_fields_device(5, dims, "cuda")
    Ud = LI.ape_smooth(Ud, steps=10, alpha=0.5).to(torch.complex64)
    U_lo = P.pack_gauge(lat, Ud, P.F32, 12)
    U_hi = P.pack_gauge(lat, Ud, P.F64, 12)  # the FP32 values, promoted
    b = P.pack_spinor(lat, psid, P.F64, P.EVEN)
    del psid
    F, st, x, X, Y = P.solve_and_force(b, U_hi, U_lo, kappa, tol=1e-10)
    assert st.status == 0 and st.true_residual <= 1e-10
    t1 = P.new_spinor(lat, P.F64, P.EVEN)
    t2 = P.new_spinor(lat, P.F64, P.EVEN)
    tmp = P.new_spinor(lat, P.F64, P.ODD)
    P.mhat(t1, x, tmp, U_hi, kappa)
    P.mhat(t2, t1, tmp, U_hi, kappa, dagger=True)
    P.axpby(1.0, b, -1.0, t2)
    assert np.sqrt(P.norm2(t2) / P.norm2(b)) <= 1.0001e-10
    del t1, t2, tmp
    Xc = P.unpack_spinor(X)
    Yc = P.unpack_spinor(Y)
    Uc = P.unpack_gauge(U_lo)  # the links the kernels see (row 2 rebuilt)
    Fc = P.unpack_gauge(F, dtype=torch.complex64)
    # the recomputed fields stage by stage, each against the oracle's hop of
    # the previous GPU stage at 256 sampled sites of its parity (and corners):
    # X_o = D_oe X_e, Y_e = X_e - kappa^2 D_eo X_o, Y_o = (D_eo)^dag Y_e
    rs = np.random.default_rng(18)
    corners = np.array([[x, y, z, t] for x in (0, dims[0] - 1) for y in (0, dims[1] - 1)
                        for z in (0, dims[2] - 1) for t in (0, dims[3] - 1)])
    cand = np.concatenate([corners, np.stack([rs.integers(0, d, 1024) for d in dims], 1)])
    odd_s = cand[cand.sum(1) % 2 == 1][:256]
    even_s = cand[cand.sum(1) % 2 == 0][:256]
    gx, gy, gu = DeviceGather(Xc), DeviceGather(Yc), DeviceGather(Uc)

    def at(field, st):
        return field[st[:, 3], st[:, 2], st[:, 1], st[:, 0]].cpu().numpy().astype(np.complex128)

    for name, got, want in (
            ("X_o", at(Xc, odd_s), dirac.dhop_at(gx, gu, odd_s)),
            ("Y_e", at(Yc, even_s), at(Xc, even_s) - kappa ** 2 * dirac.dhop_at(gx, gu, even_s)),
            ("Y_o", at(Yc, odd_s), dirac.dhop_at(gy, gu, odd_s, dagger=True))):
        assert rel(got, want) < 2e-6, name
        assert site_rel(got, want) < 2e-6, name
    rng = np.random.default_rng(12)
    links = np.stack([rng.integers(0, d, 128) for d in dims] + [rng.integers(0, 4, 128)], 1)
    links[0] = [0, 0, 0, dims[3] - 1, 3]
    links[1] = [dims[0] - 1, dims[1] - 1, dims[2] - 1, dims[3] - 1, 0]
    G = force.link_gradient_at(DeviceGather(Xc), DeviceGather(Yc), None, 2 * kappa ** 2, links)
    idx = tuple(torch.as_tensor(links[:, k]) for k in (3, 2, 1, 0, 4))
    ul = Uc[idx].cpu().numpy()
    want = force.su3_force_at(G, ul)
    got = Fc[idx].cpu().numpy().astype(np.complex128)
    assert rel(got, want) < 2e-6
    assert site_rel(got, want, per=9) < 2e-6


# Large lattices reach the force kernel's traversal orders: 32^4 (z-slab
# bricks), 32x32x36x16 (bricks sized by the L2 budget) and 18x18x42x40
# (plain order, ragged last tile).
@pytest.mark.slow
@pytest.mark.parametrize("dims", [(32, 32, 32, 32), (32, 32, 36, 16), (18, 18, 42, 40)])
@pytest.mark.parametrize("prec,link", [(P.F64, 18), (P.F32, 12)])
def test_force_large_sampled(dims, prec, link):
    """Force and raw gradient on large lattices against the oracle's link
    formula at 128 sampled links, including links that cross the last slice
    in every direction (FP64 arithmetic on the stored inputs)."""
    from tests.gpu_helpers import DeviceGather
    lat = P.Lattice(dims)
    Ud, Xd = LI.workload_fields_device(40, dims, "cuda")
    _, Yd = LI.workload_fields_device(41, dims, "cuda")
    tdt = torch.complex64 if prec == P.F32 else torch.complex128
    Uf = P.pack_gauge(lat, Ud.to(tdt), prec, link)
    Xf = P.pack_spinor(lat, Xd.to(tdt), prec)
    Yf = P.pack_spinor(lat, Yd.to(tdt), prec)
    c0 = 0.29
    G = P.fermion_force(Xf, Yf, Uf, c0, mode=1)
    F = P.fermion_force(Xf, Yf, Uf, c0, mode=0)
    Xc, Yc = P.unpack_spinor(Xf), P.unpack_spinor(Yf)
    Uc = P.unpack_gauge(Uf)  # the links the kernel sees (row 2 rebuilt)
    rng = np.random.default_rng(13)
    picked = np.stack([rng.integers(0, d, 128) for d in dims] + [rng.integers(0, 4, 128)], 1)
    for mu in range(4):
        picked[mu] = [d - 1 for d in dims] + [mu]
        picked[4 + mu] = [0, 0, 0, 0, mu]
    want_g = force.link_gradient_at(DeviceGather(Xc), DeviceGather(Yc), None, c0, picked)
    idx = tuple(torch.as_tensor(picked[:, k]) for k in (3, 2, 1, 0, 4))
    want_f = force.su3_force_at(want_g, Uc[idx].cpu().numpy().astype(np.complex128))
    tol = 2e-6 if prec == P.F32 else 1e-13
    got_g = P.unpack_gauge(G)[idx].cpu().numpy().astype(np.complex128)
    got_f = P.unpack_gauge(F)[idx].cpu().numpy().astype(np.complex128)
    assert rel(got_g, want_g) < tol
    assert rel(got_f, want_f) < tol


@pytest.mark.parametrize("inner", [(P.F64, 18), (P.F32, 12)])
def test_normal_solve_vjp_vs_oracle(inner):
    """Gradients through the solve (adjoint solve + force kernel) against
    the oracle's vector-Jacobian product."""
    dims = (8, 4, 4, 8)
    lat = P.Lattice(dims)
    U, b = LI.workload_fields(37, dims)
    b = dirac.project(b, 0)
    g = dirac.project(LI.gaussian_spinor(np.random.default_rng(38), dims), 0)
    tb = dev(b).requires_grad_(True)
    tU = dev(U).requires_grad_(True)
    x = P.normal_solve(tb, tU, KAPPA, lat, *inner, tol=1e-13)
    x.backward(dev(g))
    xo, _, _ = solver.solve_normal(b, U, KAPPA, tol=1e-14)
    lam, G = force.normal_solve_vjp(xo, g, U, KAPPA, tol=1e-14)
    assert rel(host(x), xo) < 1e-11
    assert rel(host(tb.grad), lam) < 1e-11
    assert rel(host(tU.grad), G) < 1e-10


def test_normal_solve_gradcheck_2x4():
    dims = (2, 2, 2, 2)
    lat = P.Lattice(dims)
    U, b = LI.workload_fields(39, dims)
    tb = dev(dirac.project(b, 0)).requires_grad_(True)
    tU = dev(U).requires_grad_(True)
    f = lambda bb, uu: P.normal_solve(bb, uu, KAPPA, lat, P.F64, P.LINK18, tol=1e-13)  # noqa: E731
    assert torch.autograd.gradcheck(f, (tb, tU), eps=1e-5, atol=1e-6, rtol=1e-5)


@pytest.mark.parametrize("wants", [(True, False), (False, True), (True, True)])
def test_autograd_saved_fields(wants):
    """The backward pass reads the fields packed by the forward pass: each
    combination of wanted gradients gives the bits of the full one, through
    saved-tensor hooks too, and a change of psi or U in between is refused."""
    dims = (6, 4, 2, 6)
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields(36, dims)
    g = dev(LI.gaussian_spinor(np.random.default_rng(37), dims))

    def run(wants):
        a = dev(psi).requires_grad_(wants[0])
        b = dev(U).requires_grad_(wants[1])
        return a, b, P.wilson_matrix(a, b, KAPPA, lat, P.F64, P.LINK12)

    a, b, phi = run((True, True))
    phi.backward(g)
    full = (a.grad, b.grad)
    with torch.autograd.graph.save_on_cpu():
        a, b, phi = run(wants)
    phi.backward(g, retain_graph=True)
    phi.backward(g)
    for got, want, asked in zip((a.grad, b.grad), full, wants):
        assert (got is None) if not asked else torch.equal(got, 2 * want)
    for which in (0, 1):
        a, b, phi = run(wants)
        with torch.no_grad():
            (a, b)[which].mul_(2)
        with pytest.raises(RuntimeError):
            phi.backward(g)
