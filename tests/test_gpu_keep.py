"""Memory that a chain of differentiated operators holds until its backward
pass: the packed fields kept beside psi and U stay within their bound, and the
gradients are the same bits whether an application kept its fields or not."""

import pytest
import torch

import lattice_inputs as LI
import paper_2001_07557_amd as P

pytestmark = pytest.mark.gpu

KAPPA = 0.11


def chain(lat, psi, U, n):
    for _ in range(n):
        psi = P.wilson_matrix(psi, U, KAPPA, lat, P.F64, P.LINK18)
    return psi


def test_a_long_chain_stays_within_the_bound():
    dims, n = (24, 24, 24, 24), 12
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields_device(41, dims, "cuda")
    spinor = psi.numel() * psi.element_size()
    packed = lat.gauge_bytes(P.F64, 18) + lat.spinor_bytes(P.F64, P.FULL)
    bound = 1 << 30
    assert n * packed > 2 * bound
    psi.requires_grad_(True)
    U.requires_grad_(True)
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    out = chain(lat, psi, U, n)
    held = torch.cuda.memory_allocated() - before
    # every result is the next application's psi; 2 MiB for rounding
    assert held <= n * spinor + bound + (2 << 20), held
    g = torch.ones_like(psi)
    long = torch.autograd.grad(out, (psi, U), g)
    del out
    # the same chain by itself, one application at a time, each within the bound
    with torch.no_grad():
        steps = [psi]
        for _ in range(n - 1):
            steps.append(chain(lat, steps[-1], U, 1))
    gU = 0
    for x in reversed(steps):
        x = x.detach().requires_grad_(True)
        g, step = torch.autograd.grad(chain(lat, x, U, 1), (x, U), g)
        gU = step + gU
    assert torch.equal(long[0], g)
    assert torch.equal(long[1], gU) or (long[1] - gU).abs().max() <= 1e-14 * gU.abs().max()
