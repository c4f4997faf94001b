"""Fields of more 16-byte words than one dimension of a launch can count work
items (2^32): accepted by every kernel that walks a field word by word."""

import pytest
import torch

import paper_2001_07557_amd as P

pytestmark = pytest.mark.gpu


def test_axpby_beyond_2_to_32_words():
    lat = P.Lattice((128, 128, 148, 148))
    n = lat.spinor_bytes(P.F64, P.FULL)
    assert n // 16 > 1 << 32
    torch.cuda.empty_cache()
    y = P.new_spinor(lat, P.F64, P.FULL, zero=False)
    v = y.buf[:n].view(torch.float64)
    v.fill_(2.0)
    P.axpby(0.5, y, 0.25, y)  # each word is read before it is written
    step = 1 << 28
    for at in range(0, v.numel(), step):
        right = torch.all(v[at:at + step] == 1.5).item()
        assert right, at
    del v, y
    torch.cuda.empty_cache()


def test_same_precision_convert_beyond_2_to_32_words():
    lat = P.Lattice((128, 128, 148, 148))
    n = lat.spinor_bytes(P.F64, P.FULL)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 2 * n + (8 << 30):
        pytest.skip("two fields of 69 GB do not fit")
    src, dst = (P.new_spinor(lat, P.F64, P.FULL, zero=False) for _ in range(2))
    src.buf[:n].view(torch.float64).fill_(2.0)
    dst.buf.fill_(0xFF)
    P.convert(dst, src)
    v, step = dst.buf[:n].view(torch.float64), 1 << 28
    for at in range(0, v.numel(), step):
        right = torch.all(v[at:at + step] == 2.0).item()
        assert right, at
    del v, src, dst
    torch.cuda.empty_cache()


def test_shift_beyond_2_to_32_words():
    """One word per thread: a constant field shifted in x, whose boundary is
    periodic, is the same field."""
    lat = P.Lattice((128, 128, 148, 148))
    n = lat.spinor_bytes(P.F64, P.FULL)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 2 * n + (8 << 30):
        pytest.skip("two fields of 69 GB do not fit")
    src, dst = (P.new_spinor(lat, P.F64, P.FULL, zero=False) for _ in range(2))
    src.buf[:n].view(torch.float64).fill_(3.0)
    dst.buf.fill_(0xFF)
    P.cshift(dst, src, 0, 1)
    v, step = dst.buf[:n].view(torch.float64), 1 << 28
    for at in range(0, v.numel(), step):
        right = torch.all(v[at:at + step] == 3.0).item()
        assert right, at
    del v, src, dst
    torch.cuda.empty_cache()


@pytest.mark.parametrize("vl", [64, 96])
def test_rotation_beyond_2_to_32_elements(vl):
    n = (1 << 32) // 192 * 192 + 192 * 1000
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 2 * 8 * n + (12 << 30):
        pytest.skip("two arrays of 34 GB do not fit")
    x = torch.arange(vl, dtype=torch.float64, device="cuda").repeat(n // vl).view(-1, vl)
    out = torch.full_like(x, -1.0)
    P.split_rotate(out, x, 1, 3)
    want = torch.arange(vl, dtype=torch.float64, device="cuda").roll(-3)
    step = 1 << 21
    for at in range(0, out.shape[0], step):
        right = torch.all(out[at:at + step] == want).item()
        assert right, at
    del x, out
    torch.cuda.empty_cache()
