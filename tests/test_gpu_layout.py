"""Layout conversion at the edges of its blocks, against the layout written
out with plain index arithmetic: values move, so every bit must agree."""

import numpy as np
import pytest
import torch

import paper_2001_07557_amd as P
from paper_2001_07557_amd import lqcd as L
from tests.gpu_helpers import dev, host

pytestmark = pytest.mark.gpu

# checkerboard sites per parity: 8, 32, 72, 120 (ragged second tile),
# 144 (2.25 tiles), 528, 2048
DIMS = [(2, 2, 2, 2), (2, 4, 2, 4), (6, 6, 2, 2), (10, 2, 6, 2), (6, 4, 2, 6), (22, 6, 4, 2), (8, 8, 8, 8)]
REALS = {P.F64: np.float64, P.F32: np.float32}
PER = {P.F64: 1, P.F32: 2}  # complexes per 16-byte word


def parity(dims):
    lx, ly, lz, lt = dims
    t, z, y, x = np.meshgrid(*(np.arange(n) for n in (lt, lz, ly, lx)), indexing="ij")
    return ((x + y + z + t) % 2).reshape(-1)


def words(block, prec):
    """[64 sites, n] complex -> the block's bytes as 64-lane words."""
    real = REALS[prec]
    per = PER[prec]
    out = []
    for k in range(0, block.shape[1], per):
        w = block[:, k:k + per]
        out.append(np.ascontiguousarray(w).view(real).reshape(-1))
    return np.concatenate(out)


def tiles(field, dims, prec, p):
    """Half field of parity p: (bytes as reals, which of them are padding)."""
    f = field.reshape(-1, field.shape[-1])[parity(dims) == p]
    f = f.astype(np.complex64 if prec == P.F32 else np.complex128)
    pad = -len(f) % 64
    used = np.concatenate([np.ones(len(f)), np.zeros(pad)]).astype(bool)
    f = np.concatenate([f, np.zeros((pad, f.shape[1]), f.dtype)])
    data, mask = [], []
    for s in range(0, len(f), 64):
        data.append(words(f[s:s + 64], prec))
        m = np.repeat(used[s:s + 64, None], f.shape[1], 1).astype(f.dtype)
        mask.append(words(m + 1j * m, prec) != 0)
    return np.concatenate(data), np.concatenate(mask)


def draw(rng, shape, dtype):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(dtype)


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec", [P.F64, P.F32])
@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
def test_spinor_layout_bits(dims, prec, dtype):
    lat = P.Lattice(dims)
    psi = draw(np.random.default_rng(5), lat.spinor_shape(), dtype)
    for subset in (P.EVEN, P.ODD, P.FULL):
        halves = (0, 1) if subset == P.FULL else (subset,)
        parts = [tiles(psi.reshape(-1, 12), dims, prec, p) for p in halves]
        f = P.pack_spinor(lat, dev(psi), prec, subset)
        got = host(f.buf)[:lat.spinor_bytes(prec, subset)].view(REALS[prec])
        want, used = (np.concatenate(x) for x in zip(*parts))
        assert np.array_equal(got[used], want[used]), subset
        # back: sites of the other parity keep what they held
        out = torch.full(lat.spinor_shape(), 7.0 + 3.0j, dtype=dev(psi).dtype, device="cuda")
        P.unpack_spinor(f, out=out)
        inside = np.isin(parity(dims), halves).reshape(psi.shape[:4])
        stored = psi.astype(np.complex64).astype(dtype) if prec == P.F32 else psi
        assert np.array_equal(host(out)[inside], stored[inside])
        assert np.all(host(out)[~inside] == 7.0 + 3.0j)


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec,link", [(P.F64, 18), (P.F64, 12), (P.F32, 18), (P.F32, 12)])
@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
def test_gauge_layout_bits(dims, prec, link, dtype):
    lat = P.Lattice(dims)
    U = draw(np.random.default_rng(6), lat.links_shape(), dtype)
    n = link // 2
    f = P.pack_gauge(lat, dev(U), prec, link)
    got = host(f.buf)[:lat.gauge_bytes(prec, link)].view(REALS[prec])
    ntiles = -(-lat.half_volume // 64)
    # [parity][tile][mu][n complexes as words][64 sites]; of nine FP32
    # complexes the last is a word of 8 bytes
    got = got.reshape(2, ntiles, 4, n * 2 * 64)
    for p in (0, 1):
        for mu in range(4):
            u = U[..., mu, :, :].reshape(-1, 9)[:, :n]
            head = n // PER[prec] * PER[prec]
            a, am = tiles(u[:, :head], dims, prec, p)
            a, am = a.reshape(ntiles, -1), am.reshape(ntiles, -1)
            if head < n:
                b, bm = tiles(np.concatenate([u[:, head:]] * 2, 1), dims, prec, p)
                b, bm = (x.reshape(ntiles, 64, 2, 2)[:, :, 0].reshape(ntiles, -1) for x in (b, bm))
                a, am = np.concatenate([a, b], 1), np.concatenate([am, bm], 1)
            assert np.array_equal(got[p, :, mu][am], a[am]), (p, mu)
    if link == 18:
        back = host(P.unpack_gauge(f, dtype=dev(U).dtype))
        assert np.array_equal(back, U.astype(np.complex64).astype(dtype) if prec == P.F32 else U)


# ragged and whole tiles, and the smallest lattice of the blocked tile order
OUT_DIMS = [(2, 2, 2, 2), (6, 4, 2, 6), (22, 6, 4, 2), (8, 8, 8, 8), (16, 16, 16, 64)]


@pytest.mark.parametrize("dims", OUT_DIMS)
@pytest.mark.parametrize("prec,link", [(P.F64, 18), (P.F64, 12), (P.F32, 18), (P.F32, 12)])
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_canonical_results_equal_unpacked_ones(dims, prec, link, dtype):
    """The operator and the link gradient written as canonical arrays by
    their own kernels: the bits of the internal result, unpacked."""
    lat = P.Lattice(dims, (-1, 1, 1, -1))
    rng = np.random.default_rng(7)
    U = P.pack_gauge(lat, dev(draw(rng, lat.links_shape(), np.complex128)), prec, link)
    x, y = (P.pack_spinor(lat, dev(draw(rng, lat.spinor_shape(), np.complex128)), prec) for _ in range(2))
    out = P.new_spinor(lat, prec, P.FULL)
    for dagger in (False, True):
        want = P.unpack_spinor(P.wilson(out, x, U, 0.11, dagger), dtype=dtype)
        assert torch.equal(L.wilson_canonical(x, U, 0.11, dtype, dagger), want)
    add = P.fermion_force(y, x, U, 0.3, mode=1)
    for mode in (0, 1) + ((2,) if link == 12 else ()):
        want = P.unpack_gauge(P.fermion_force(x, y, U, 0.7, mode=mode), dtype=dtype)
        assert torch.equal(L.fermion_force_canonical(x, y, U, 0.7, mode, dtype), want)
        both = P.new_gauge(lat, prec, P.LINK18)
        both.buf.copy_(add.buf)
        want = P.unpack_gauge(P.fermion_force(x, y, U, 0.7, mode=mode, out=both, accumulate=True), dtype=dtype)
        assert torch.equal(L.fermion_force_canonical(x, y, U, 0.7, mode, dtype, add=add), want)
