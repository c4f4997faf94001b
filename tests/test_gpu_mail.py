"""Sums that reach the host through posted slots: a call that gives up leaves
nothing behind for the next one."""

import ctypes

import pytest
import torch

import paper_2001_07557_amd as P
from paper_2001_07557_amd import _lib

pytestmark = pytest.mark.gpu


def field(lat, value):
    f = P.new_spinor(lat, P.F64, P.FULL)
    f.buf[:lat.spinor_bytes(P.F64, P.FULL)].view(torch.float64).fill_(value)
    return f


def norm2(lib, f, ws, res):
    return lib.lqcd_norm2(f.lattice.ref(), f.subset, f.ptr, f.prec, ws.data_ptr(), res,
                          torch.cuda.current_stream().cuda_stream)


def test_sum_after_a_call_that_gave_up():
    """An error that an earlier HIP call of the thread left unread makes
    lqcd_norm2 fail after its launches; the next call, on another field, must
    not take the first one's sum, whose post is still to come."""
    lib = _lib.load()
    lat = P.Lattice((8, 8, 8, 8))
    a, b = field(lat, 1.0), field(lat, 3.0)
    ws = [torch.empty(lib.lqcd_reduce_workspace_bytes(lat.ref(), P.FULL), dtype=torch.uint8, device="cuda")
          for _ in range(2)]
    res = [(ctypes.c_double * 1)() for _ in range(2)]
    assert P.norm2(a) == 24.0 * lat.volume and P.norm2(b) == 9.0 * 24.0 * lat.volume
    torch.cuda.synchronize()
    torch.cuda._sleep(10_000_000)  # the stream is busy while both calls are made
    lib.hipSetDevice(-1)  # an invalid argument: refused, and the refusal left unread
    first = norm2(lib, a, ws[0], res[0])
    second = norm2(lib, b, ws[1], res[1])
    torch.cuda.synchronize()
    assert first == -2 and second == 0
    assert res[1][0] == 9.0 * 24.0 * lat.volume


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (16, 16, 16, 16)])
@pytest.mark.parametrize("busy", [0, 1_000_000])
def test_sums_synchronise_the_stream(dims, busy):
    """lqcd_dot and lqcd_norm2 return when the stream has drained."""
    lat = P.Lattice(dims)
    f = field(lat, 1.0)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        for call in (lambda: P.norm2(f), lambda: P.dot(f, f).real):
            for _ in range(20):
                if busy:
                    torch.cuda._sleep(busy)
                assert call() == 24.0 * lat.volume
                assert stream.query()
