"""The solver's sums at the sizes where they are made another way: up to
1024 partials each block of the last hop sums them itself, above it the hop
before sums them in groups, and above 16384 the direction update is given
group sums too.  A wrong sum is a wrong step: the solve would take more
iterations than the FP64 one of the same system, or never converge."""

import pytest

import lattice_inputs as LI
import paper_2001_07557_amd as P

pytestmark = pytest.mark.gpu

# tiles per parity: 1, 3, 130 (two groups' runs of unequal length), 1024,
# 1088, 16384, 16896
DIMS = [(2, 4, 4, 4), (6, 6, 6, 2), (8, 8, 10, 26), (16, 16, 16, 32), (16, 16, 16, 34), (32, 32, 32, 64),
        (32, 32, 32, 66)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec", [P.F64, P.F32, P.F16])
def test_solve_at_the_edges_of_the_sums(dims, prec):
    kappa, tol = 0.12, 1e-10
    lat = P.Lattice(dims)
    U, psi = LI.workload_fields_device(12, dims, "cuda")
    hi = P.pack_gauge(lat, U, P.F64, 12)
    lo = hi if prec == P.F64 else P.pack_gauge(lat, U, prec, 12)
    b = P.pack_spinor(lat, psi, P.F64, P.EVEN)
    del U, psi
    x, mx, ax = (P.new_spinor(lat, P.F64, P.EVEN) for _ in range(3))
    tmp = P.new_spinor(lat, P.F64, P.ODD)
    ref = P.cg_solve(P.new_spinor(lat, P.F64, P.EVEN), b, hi, hi, kappa, tol=tol)
    st = P.cg_solve(x, b, hi, lo, kappa, tol=tol, reliable_every=0)
    P.mhat(mx, x, tmp, hi, kappa)
    P.mhat(ax, mx, tmp, hi, kappa, dagger=True)
    bb = P.norm2(b)
    P.axpby(1.0, b, -1.0, ax)
    assert (P.norm2(ax) / bb) ** 0.5 <= tol
    # binary16 restarts its recurrence at every tenfold fall
    assert st.iterations <= ref.iterations * (1.0 if prec == P.F64 else 1.1 if prec == P.F32 else 1.6) + 2
    # from a guess: the residual of the guess starts the iteration
    P.axpby(0.999, x, 0.0, mx)
    st2 = P.cg_solve(mx, b, hi, lo, kappa, tol=tol)
    assert st2.true_residual <= tol and 0 < st2.iterations <= st.iterations


def test_solves_on_threads_and_streams():
    """Solves that run at once, each on its own thread and stream, get their
    own sums: the bits of the same solve alone."""
    import threading

    import torch
    dims, kappa, jobs = (8, 8, 8, 8), 0.12, 4
    lat = P.Lattice(dims)

    def solve(seed):
        U, psi = LI.workload_fields_device(seed, dims, "cuda")
        hi, lo = P.pack_gauge(lat, U, P.F64, 12), P.pack_gauge(lat, U, P.F32, 12)
        b, x = P.pack_spinor(lat, psi, P.F64, P.EVEN), P.new_spinor(lat, P.F64, P.EVEN)
        st = P.cg_solve(x, b, hi, lo, kappa)
        return st.iterations, st.true_residual, x.buf.cpu()

    alone = [solve(20 + i) for i in range(jobs)]
    got = [[] for _ in range(2 * jobs)]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                got[i].append(solve(20 + i % jobs))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2 * jobs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i, results in enumerate(got):
        assert len(results) == 3
        for n, res, x in results:
            assert (n, res) == alone[i % jobs][:2] and torch.equal(x, alone[i % jobs][2])
