"""Launches of more work items than one counts (2^32) are refused before they
reach the device, not cut short (host only: the pointers are never read)."""

import ctypes

import pytest
import torch

import paper_2001_07557_amd as P
from paper_2001_07557_amd import _lib
from paper_2001_07557_amd.lqcd import EINVAL


@pytest.mark.skipif(torch.cuda.is_available(), reason="made-up pointers: on a machine without a GPU only")
def test_operator_beyond_a_launch_is_refused():
    lib = _lib.load()
    out, inp, U = (ctypes.c_void_p(i << 40) for i in (1, 2, 3))
    for dims in ((256, 128, 128, 128), (82, 10, 10, 65536)):
        big = P.Lattice(dims)
        assert big.volume >= 1 << 29
        for fn in (lib.lqcd_dslash, lib.lqcd_dslash_dagger):
            assert fn(big.ref(), out, inp, None, U, 1.0, 0.0, P.F32, 12, None) == EINVAL
