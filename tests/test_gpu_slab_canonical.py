"""Canonical results of launches in slab order, whose grid has blocks beyond
the last tile and whose ragged tile is not the last block's: the operator and
the link gradient written by their own kernels against the internal results,
unpacked; no byte outside the array is written."""

import pytest
import torch

import lattice_inputs as LI
import paper_2001_07557_amd as P
from paper_2001_07557_amd import _lib
from paper_2001_07557_amd import lqcd as L

pytestmark = pytest.mark.gpu

# a ragged last tile; whole tiles; six planes (a slab thinner than a plane)
DIMS = [(18, 18, 42, 40), (28, 28, 28, 28), (46, 46, 6, 60)]
GUARD = 1 << 16


def guarded(shape, dtype):
    """A tensor with GUARD bytes of 0xA5 on either side of it."""
    n = torch.empty(0, dtype=dtype).element_size()
    for d in shape:
        n *= d
    buf = torch.full((n + 2 * GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    return buf, buf[GUARD:GUARD + n].view(dtype).view(shape)


def untouched(buf):
    return bool((buf[:GUARD] == 0xA5).all()) and bool((buf[-GUARD:] == 0xA5).all())


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec,link", [(P.F64, 18), (P.F64, 12), (P.F32, 18), (P.F32, 12)])
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_canonical_results_in_slab_order(dims, prec, link, dtype):
    lib, lat = _lib.load(), P.Lattice(dims, (-1, 1, 1, -1))
    canon = L._canon_prec(torch.empty(0, dtype=dtype))
    U, psi = LI.workload_fields_device(61, dims, "cuda")
    Uf, x = P.pack_gauge(lat, U, prec, link), P.pack_spinor(lat, psi, prec)
    y = P.pack_spinor(lat, psi.roll(1, 0), prec)
    del U, psi
    out, stream = P.new_spinor(lat, prec, P.FULL), torch.cuda.current_stream().cuda_stream
    for dagger in (0, 1):
        want = P.unpack_spinor(P.wilson(out, x, Uf, 0.11, bool(dagger)), dtype=dtype)
        buf, res = guarded(lat.spinor_shape(), dtype)
        assert lib.lqcd_dslash_canonical(lat.ref(), res.data_ptr(), canon, x.ptr, x.ptr, Uf.ptr, -0.11, 1.0,
                                         dagger, prec, link, stream) == 0
        same = torch.equal(res, want)
        assert same and untouched(buf), dagger
    del out, res, buf, want
    add = P.fermion_force(y, x, Uf, 0.3, mode=1)
    for mode in (0, 1) + ((2,) if link == 12 else ()):
        for with_add in (False, True):
            F = P.new_gauge(lat, prec, P.LINK18)
            if with_add:
                F.buf.copy_(add.buf)
            P.fermion_force(x, y, Uf, 0.7, mode=mode, out=F, accumulate=with_add)
            want = P.unpack_gauge(F, dtype=dtype)
            buf, res = guarded(lat.links_shape(), dtype)
            assert lib.lqcd_fermion_force_canonical(lat.ref(), res.data_ptr(), canon,
                                                    add.ptr if with_add else None, x.ptr, y.ptr, Uf.ptr, 0.7,
                                                    mode, prec, link, stream) == 0
            same = torch.equal(res, want)
            assert same and untouched(buf), (mode, with_add)


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 2, 6), (8, 8, 8, 8)])
@pytest.mark.parametrize("prec", [P.F64, P.F32, P.F16])
@pytest.mark.parametrize("parity", [P.EVEN, P.ODD])
def test_update_of_a_half_leaves_the_other_half(dims, prec, parity):
    """lqcd_axpby on one half of a full field: the bytes of the other half,
    and of what follows the field, stay."""
    lat = P.Lattice(dims)
    x, y = (P.new_spinor(lat, prec, P.FULL) for _ in range(2))
    for f in (x, y):
        f.buf.random_(generator=torch.Generator(device="cuda").manual_seed(9))
    for f in (x, y):
        P.pack_spinor(lat, torch.ones(lat.spinor_shape(), dtype=torch.complex128, device="cuda"), prec,
                      parity, out=f.half(parity))
    before = y.buf.clone()
    P.axpby(0.5, x.half(parity), 2.0, y.half(parity))
    hb = lat.spinor_bytes(prec, parity)
    mine = torch.zeros_like(before, dtype=torch.bool)
    mine[parity * hb:(parity + 1) * hb] = True
    kept = torch.equal(y.buf[~mine], before[~mine])
    assert kept
    got = P.unpack_spinor(y.half(parity))
    assert abs(got.sum().real.item() - 2.5 * 12 * lat.half_volume) <= 1e-3 * lat.half_volume
