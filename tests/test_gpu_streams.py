"""Streaming kernels at the edges of their blocks: sums and updates of fields
whose last tile is ragged, with NaN in the padding lanes (nothing may read
them into a sum), and the lane permutation where a vector straddles blocks."""

import numpy as np
import pytest
import torch

import paper_2001_07557_amd as P
from tests.gpu_helpers import dev, host

pytestmark = pytest.mark.gpu

# V/2 = 8, 72, 120, 144, 2048 (whole tiles), 272160 (more words than the grid
# takes in one step)
DIMS = [(2, 2, 2, 2), (6, 6, 2, 2), (10, 2, 6, 2), (6, 4, 2, 6), (8, 8, 8, 8), (18, 18, 42, 40)]


def poisoned(lat, psi, prec, subset):
    f = P.new_spinor(lat, prec, subset, zero=False)
    f.buf.fill_(0xFF)
    return P.pack_spinor(lat, psi, prec, subset, out=f)


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec", [P.F64, P.F32, P.F16])
@pytest.mark.parametrize("subset", [P.EVEN, P.ODD, P.FULL])
def test_sums_leave_padding_out(dims, prec, subset):
    lat = P.Lattice(dims)
    gen = torch.Generator(device="cuda").manual_seed(3)
    draw = lambda: torch.view_as_complex(torch.randn(lat.spinor_shape() + (2,), generator=gen, device="cuda",  # noqa: E731
                                                     dtype=torch.float64))
    a, b = (poisoned(lat, draw(), prec, subset) for _ in range(2))
    ra, rb = (P.unpack_spinor(f).reshape(-1) for f in (a, b))
    want = torch.sum(ra.conj() * rb).item()
    na, nb = torch.sum(ra.abs() ** 2).item(), torch.sum(rb.abs() ** 2).item()
    # products of one word in the field's arithmetic, everything above in FP64
    tol = 1e-13 if prec == P.F64 else 1e-6
    got = P.dot(a, b)
    assert abs(got - want) <= tol * (na * nb) ** 0.5
    assert got == P.dot(a, b)
    assert abs(P.norm2(a) - na) <= tol * na
    # the update, and that it leaves the sites outside the subset alone
    P.axpby(0.5, a, -1.25, b)
    upd = P.unpack_spinor(b).reshape(-1)
    exact = 0.5 * ra - 1.25 * rb
    err = (upd - exact).abs().max().item()
    assert err <= {P.F64: 1e-15, P.F32: 5e-7, P.F16: 2e-3}[prec] * exact.abs().max().item()


@pytest.mark.parametrize("vl,s", [(96, 1), (96, 8), (256, 8), (3, 1), (65, 5), (1023, 3), (1025, 1), (4096, 16)])
@pytest.mark.parametrize("nvec", [1, 7, 33])
@pytest.mark.parametrize("dtype", [np.float64, np.complex128])
def test_split_rotate_across_blocks(vl, s, nvec, dtype):
    rng = np.random.default_rng(vl + nvec)
    x = rng.standard_normal((nvec, vl)).astype(dtype)
    w = vl // s
    for r in {0, 1, w // 2, w - 1, w, -1}:
        out = torch.full((nvec, vl), 7.0, dtype=torch.from_numpy(x).dtype, device="cuda")
        P.split_rotate(out, dev(x), s, r)
        want = np.roll(x.reshape(nvec, s, w), -r, axis=2).reshape(nvec, vl)
        assert np.array_equal(host(out), want), r


def test_sums_are_refused_under_capture():
    """A result for the host cannot come from a stream that is captured: the
    call returns an error, as a copy does, and the process goes on."""
    lat = P.Lattice((4, 4, 4, 4))
    f = P.new_spinor(lat, P.F64, P.EVEN)
    assert P.norm2(f) == 0.0
    stream = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    refused = False
    with torch.cuda.stream(stream):
        g.capture_begin(capture_error_mode="thread_local")
        try:
            P.norm2(f)
        except P.LQCDError:
            refused = True
        try:
            g.capture_end()
        except RuntimeError:
            pass  # the refused call has ended the capture
    assert refused
    torch.cuda.synchronize()
    assert P.norm2(f) == 0.0
