// Conjugate gradient on the even-odd normal system A = Mhat^dag Mhat with
// reliable updates: the inner iteration runs in the storage precision of the
// sloppy gauge field (FP64, FP32 or binary16 storage with FP32 arithmetic),
// global sums are FP64 and fixed-order, and the true residual b - A x is
// recomputed in FP64 every `reliable_every` iterations, whenever a
// reduced-precision inner residual has fallen by 1/delta since the last
// update (delta below), and whenever the inner residual reaches the
// tolerance.  CG scalars live in device memory, so an iteration is a stream
// of kernels with no host round trip; the host reads the residual every few
// iterations, and every iteration once the decay so far says the tolerance
// is near, so the solve stops at the first iteration that reaches it.
//
// Per iteration five launches (four, below, on small lattices): the direction update (x += a p, p = r + b p;
// its blocks finish the |r|^2 sum and form beta themselves), four hops (the
// second leaves the |Mhat p|^2 = <p, A p> block partials, the third sums runs
// of them on the side, the fourth forms alpha from those, does r -= a A p in
// its epilogue, so A p is never stored, and leaves the |r|^2 partials).
// On small lattices (CG_FEW partials, FP64 and FP32 inner) the direction
// update is part of the first two hops and an iteration is four launches:
// 16^4 FP32 5.4 + 6.3 + 5.7 + 6.5 + 5.8 -> 7.7 + 7.2 + 5.4 + 6.7 us under the
// trace and one gap less, 4.53 -> 4.21 ms for a differentiable solve.
// Kernel times per iteration (us, trace; seven launches before, with two
// one-block scalar kernels and x updated in the fourth hop): 32^4 binary16
// inner 26 + 30 + 26 + 43 + 12.5 + 2 x 4.9 -> 26 + 30 + 26 + 35 + 23, 24^3x48
// FP32 29 + 34 + 29 + 53 + 15 + 2 x 4.8 -> 30 + 34 + 29 + 40 + 26 (the
// direction update moves 159 MB, 6.1 TB/s).

#include <chrono>
#include <cmath>
#include <utility>

#include "lqcd_internal.h"
#include "reduce.h"
#include "hop_common.h"
#include "blas.h"
#include "mail.h"

namespace lqcd {

constexpr int CG_BLOCK = 256;
constexpr int CHECK_EVERY = 10;
// A reduced-precision inner recurrence is trusted only while its residual is
// within a factor delta of the last true residual: past that point the
// computed and true residuals part (rounding of the inner precision), so a
// reliable update is taken.  delta = 0.1 for binary16 storage (unit roundoff
// 2^-11), 1e-4 for FP32 (2^-24: after that drop the rounding carried by the
// recurrence is a few 1e-3 of the residual); FP64 inner iterations need it
// only at the end.  FP32 inner to 1e-10, iterations / updates with delta =
// 1e-3, 1e-4, 1e-5: 24^3x48 links spread by 0.3 around one 46/3, 46/2, 48/2
// (8.64, 8.30, 8.61 ms), by 0.15 105/4, 105/4, 106/3, Haar links 24/3, 24/2,
// 27/2; to 1e-12 1e-3 and 1e-4 take the same or one update less.
constexpr double DELTA_F16 = 0.1;
constexpr double DELTA_F32 = 1e-4;
// A reduced-precision recurrence residual runs ahead of the true one, so the
// final reliable update is taken when it reaches tol / 2 rather than tol
// (squared: 0.25): an update taken when the recurrence first touches tol
// finds the true residual still just above it and costs a second FP64 update
// a few iterations later.
constexpr double INNER_MARGIN2 = 0.25;

// Fixed-order sum of n partials, `stride` apart, by a block of SUM_BLOCK
// threads: thread t adds entries t, t + B, t + 2B, ... in four interleaved
// chains, so that four loads are in flight.  Valid in every thread.
constexpr int SUM_BLOCK = 512;
__device__ __forceinline__ double partial_total(const double *partial, int n, int stride) {
    constexpr int B = SUM_BLOCK;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int i = threadIdx.x;
    for (; i + 3 * B < n; i += 4 * B) {
        a0 += partial[(int64_t)i * stride];
        a1 += partial[(int64_t)(i + B) * stride];
        a2 += partial[(int64_t)(i + 2 * B) * stride];
        a3 += partial[(int64_t)(i + 3 * B) * stride];
    }
    for (; i < n; i += B) a0 += partial[(int64_t)i * stride];
    double v[1] = {(a0 + a1) + (a2 + a3)};
    block_sum<1>(v);
    __shared__ double total;
    if (threadIdx.x == 0) total = v[0];
    __syncthreads();
    return total;
}

// The sum (and that of a second run of n, if given) for the host, posted or
// (no mail) left for a copy.  RESID: the sum of a recomputed residual, after
// which x has no step pending.
template <bool RESID>
__global__ __launch_bounds__(SUM_BLOCK) void cg_sum_k(const double *partial, const double *second, int n,
                                                      int stride, double *sc, Mail *mail, uint64_t count) {
    const double s = partial_total(partial, n, stride);
    double t = 0.0;
    if (second) {
        __syncthreads();
        t = partial_total(second, n, stride);
    }
    if (threadIdx.x == 0) {
        if (RESID) sc[CG_ALPHA] = 0.0;
        if (mail) {
            mail_post(mail, count, s, t);
        } else {
            sc[CG_OUT] = s;
            sc[CG_OUT + 1] = t;
        }
    }
}

// Sums of CG_GROUPS runs of n partials.
__global__ __launch_bounds__(64) void cg_groups_k(const double *partial, int n, double *groups) {
    const int per = (n + CG_GROUPS - 1) / CG_GROUPS, lo = (int)blockIdx.x * per;
    const double t = wave_total(partial + lo, n - lo < per ? n - lo : per);
    if (threadIdx.x == 0) groups[blockIdx.x] = t;
}

// x += alpha p, p_new = rs + beta p.  Every block sums the n partials of |rs|^2
// (few blocks, each over several sites per thread) and forms beta = |rs|^2 /
// |rs before|^2; the first iteration finds 0 there and takes p = rs, and so
// does a restart.
constexpr int DIR_BLOCKS = 512;
// partials beyond which they are summed into groups by a launch of their own
constexpr int CG_MANY = 16384;
// partials that every block of the last hop sums itself: 512 of them (16^4)
// take a wave eight loads, while summing groups in the hop before, where all
// of its blocks run at once, put 0.9 us on a 5.2 us launch
constexpr int CG_FEW = 1024;
template <int P>
__global__ __launch_bounds__(SUM_BLOCK) void cg_direction_k(char *p_new, const char *p, const char *rs,
                                                            char *xs, double *sc,
                                                            const double *partial, int n, int slot,
                                                            bool restart, int64_t vh) {
    using T = typename real_of<P>::type;
    const int64_t step = (int64_t)gridDim.x * SUM_BLOCK;
    int64_t s = (int64_t)blockIdx.x * SUM_BLOCK + threadIdx.x;
    cplx<T> vr[12], vp[12], vx[12];
    // the first site's words arrive while the partials are summed
    if (s < vh) {
        load_spinor<P>(rs, s, vr);
        load_spinor<P>(p, s, vp);
        load_spinor<P>(xs, s, vx);
    }
    const double old = sc[CG_RR + (slot ^ 1)];
    const T alpha = (T)sc[CG_ALPHA];
    const double rr = partial_total(partial, n, 1);
    const double b = old > 0.0 && !restart ? rr / old : 0.0;
    const T beta = (T)b;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc[CG_RR + slot] = rr;
        sc[CG_BETA] = b;
    }
    while (s < vh) {
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            vx[k] = {fmad(alpha, vp[k].re, vx[k].re), fmad(alpha, vp[k].im, vx[k].im)};
            vp[k] = {fmad(beta, vp[k].re, vr[k].re), fmad(beta, vp[k].im, vr[k].im)};
        }
        store_spinor<P>(xs, s, vx);
        store_spinor<P>(p_new, s, vp);
        s += step;
        if (s < vh) {
            load_spinor<P>(rs, s, vr);
            load_spinor<P>(p, s, vp);
            load_spinor<P>(xs, s, vx);
        }
    }
}

// x64 += xs + alpha p (the step of the last iteration is still pending; the
// sum is rounded to the inner precision's storage like every step before it,
// whose loss the residual then holds along p, the direction that is kept),
// xs = 0.
template <int P>
__global__ __launch_bounds__(CG_BLOCK) void cg_fold_k(char *x64, char *xs, const char *p, const double *sc,
                                                      int64_t vh) {
    using T = typename real_of<P>::type;
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= vh) return;
    const T alpha = (T)sc[CG_ALPHA];
    cplx<double> vx[12];
    cplx<T> v[12], vp[12];
    load_spinor<LQCD_F64>(x64, s, vx);
    load_spinor<P>(xs, s, v);
    load_spinor<P>(p, s, vp);
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = {fmad(alpha, vp[k].re, v[k].re), fmad(alpha, vp[k].im, v[k].im)};
    round_stored<P>(v);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        vx[k] = {vx[k].re + (double)v[k].re, vx[k].im + (double)v[k].im};
        v[k] = {0, 0};
    }
    store_spinor<LQCD_F64>(x64, s, vx);
    store_spinor<P>(xs, s, v);
}

// Inner start from a zero guess: rs = b rounded to the inner precision, with
// one |rs as stored|^2 partial per tile, and xs = p = 0.
template <int P>
__global__ __launch_bounds__(CG_BLOCK) void cg_start_k(char *rs, char *xs, char *p, const char *b,
                                                       double *partial, int64_t vh) {
    using T = typename real_of<P>::type;
    const int64_t s = (int64_t)blockIdx.x * CG_BLOCK + threadIdx.x;
    double n = 0.0;
    if (s < vh) {
        cplx<double> vb[12];
        cplx<T> v[12];
        load_spinor<LQCD_F64>(b, s, vb);
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = {(T)vb[k].re, (T)vb[k].im};
        n = (double)store_spinor<P>(rs, s, v, true);
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = {0, 0};
        store_spinor<P>(xs, s, v);
        store_spinor<P>(p, s, v);
    }
    n = wave_sum(n);
    if ((threadIdx.x & 63) == 0 && s < vh) partial[s >> TILE_SHIFT] = n;
}

// ---------------------------------------------------------------------------
// host side of the solver
// ---------------------------------------------------------------------------

struct CGWork {
    char *xs, *rs, *te, *to;          // inner precision
    char *p[2];                       // this and the next direction
    char *te64, *to64;                // FP64 (those of an FP64 inner solve)
    double *partial;                  // of |rs|^2, one per tile
    // one per tile of <p, A p>, or of a recomputed |r|^2, or per block of an
    // FP64 norm; and of runs of them
    double *pap, *groups;
    double *sc;
    size_t bytes;
};

static size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

static CGWork cg_layout(const Geom &g, int prec, char *base) {
    CGWork w{};
    const size_t hb = align256(half_spinor_bytes(g, prec));
    const size_t hb64 = align256(half_spinor_bytes(g, LQCD_F64));
    size_t off = 0;
    auto take = [&](size_t n) {
        char *p = base ? base + off : nullptr;
        off += align256(n);
        return p;
    };
    w.xs = take(hb);
    w.rs = take(hb);
    w.p[0] = take(hb);
    w.te = take(hb);
    w.to = take(hb);
    // one FP64 field for the sums and, behind them, the second direction of a
    // reduced inner precision; an FP64 inner solve has the second direction in
    // the FP64 temporaries' place, which are its own
    char *scratch = take(hb64);
    char *t64[2] = {take(hb64), take(hb64)};
    const int64_t tiles = hop_partials(g, 1), norms = 4 * reduce_blocks(g, 1);
    w.partial = (double *)take(sizeof(double) * tiles);
    w.sc = (double *)take(sizeof(double) * CG_SCALARS);
    if (base) {
        w.groups = (double *)scratch;
        w.pap = w.groups + CG_GROUPS;
        // (sums: at most 128 + 4 per tile of the 1536 doubles per tile)
        w.p[1] = prec == LQCD_F64 ? t64[0]
                                  : scratch + align256(sizeof(double) * (CG_GROUPS + (tiles > norms ? tiles : norms)));
        w.te64 = prec == LQCD_F64 ? w.te : t64[0];
        w.to64 = prec == LQCD_F64 ? w.to : t64[1];
    }
    w.bytes = off;
    return w;
}

// Iterations the inner residual rr still needs to reach target when log(rr)
// falls by -rate per iteration (rate < 0; rate = 0: not known yet).
static int iterations_left(double rr, double rate, double target) {
    if (!(rr > target)) return 0;
    if (!(rate < 0.0)) return 1 << 20;
    const double n = std::ceil(std::log(target / rr) / rate);
    return n > (double)(1 << 20) ? 1 << 20 : (int)n;
}

// Iterations until the next host read: CHECK_EVERY while the tolerance is
// far, fewer as it nears, one once it is about an iteration away, so the
// solve stops at the first iteration whose residual reaches it instead of up
// to CHECK_EVERY - 1 later.
static int read_gap(int left) {
    const int n = (int)(0.7 * left);
    return n < 1 ? 1 : n > CHECK_EVERY ? CHECK_EVERY : n;
}

// A drift-triggered reliable update is put off while the tolerance is
// predicted this close (in iterations): the final update follows soon, and
// reading the residual every iteration near the end would otherwise add an
// FP64 update a few iterations before the last one (at 32^4 FP32 inner:
// three updates instead of two).  It is put off only until the inner
// residual is found, at a read, to have fallen DRIFT_HARD (squared: 1e-4, a
// further factor 100) below the drift threshold: without that bound an 8^4
// FP32-inner solve to 1e-12, whose recurrence keeps predicting the end, took
// 300 iterations instead of under 200 (with a threshold of 1e-3).  With the
// threshold of 1e-4 the bound is 1e-6, and 1e-2 in its place (1e-5) changes
// no solve by more than one update: 50 systems of 36 to 1400 FP64 iterations, to
// 1e-10 and 1e-12, take 0 to 9% more iterations with FP32 inner than FP64 either
// way (Haar links 8^4 kappa 0.24 1403 -> 1444 and 1634 -> 1669; kappa 0.22 267
// -> 276 and 321 -> 329; 12^4 spread by 0.4 201 -> 206 and 240 -> 254), and so
// with a threshold of 1e-3, at one or two updates more.  binary16 inner solves, whose drift rule fires at every
// tenfold fall, take every drift update (put off, the 32^4 solve needed 55
// iterations instead of 46).
constexpr int DRIFT_DEFER = CHECK_EVERY;
constexpr double DRIFT_HARD = 1e-4;
// A reliable update keeps p while the recomputed residual agrees with the
// recurrence's, and restarts from p = r where it is RESTART times larger
// (squared norms): between two host reads a binary16 recurrence can fall a
// thousand times below the true residual, beta = |r true|^2 / |r before|^2
// then weighs the old p a hundredfold, and the solve crawls.  Measured
// (iterations / updates to 1e-10, binary16 inner, p always kept -> 1.2): Haar
// links 8^4 761/9 -> 29/4; links spread by 0.4 around one 16^4 63/7 -> 37/5;
// by 0.3 24^3x48 50/6 -> 46/5 (7.41 -> 6.60 ms), 32^4 50/6 -> 46/5 (10.6 ->
// 9.5 ms); by 0.2 75/8 either way.  1.02 restarts too often (48 to 50
// iterations by 0.3), 1.5 and 2 miss the cases by 0.3, 16 those by 0.4.
constexpr double RESTART = 1.2;

struct Solver {
    Geom g;
    hipStream_t st;
    double kappa;
    int prec, link;
    const char *U;
    int link64;
    const char *U64;
    CGWork w;
    MailSlot mail;

    int hop(int out_par, char *out, const char *in, const char *y, double alpha, bool dag, int pr,
            int lk, const char *U_, double *partial, int cg = CG_NONE, int slot = 0, const char *rhs = nullptr,
            bool restart = false) {
        HopArgs a{};
        a.cg = cg;
        a.slot = slot;
        a.sc = w.sc;
        a.groups = w.groups;
        a.rhs = rhs;
        a.stored = w.partial;
        const int n = (int)hop_partials(g, 1);
        const int per = (n + CG_GROUPS - 1) / CG_GROUPS;
        a.n_groups = (n + per - 1) / per;
        a.sums = cg == CG_PRE || n <= CG_FEW ? w.pap : w.groups;
        a.n_sums = cg == CG_PRE || n <= CG_FEW ? n : a.n_groups;
        if (cg == CG_DIR_IN) a.sums = w.partial;  // n <= CG_FEW
        a.restart = restart ? 1 : 0;
        a.p_old = w.p[0];
        a.p_new = w.p[1];
        a.x = w.xs;
        a.g = g;
        a.U = U_;
        a.alpha = alpha;
        a.beta = 1.0;
        a.par0 = out_par;
        a.out[out_par] = out;
        a.in[out_par] = in;
        a.y[out_par] = y;
        a.partial = partial;
        return hop_launch(a, pr, lk, dag, 1, st);
    }

    // One inner iteration: the direction update from the |rs|^2 partials of
    // the step before (a launch of its own, or inside the first two hops),
    // te = Mhat p with the <p, A p> = |Mhat p|^2 partials, then Mhat^dag te =
    // A p formed inside the last hop, which updates rs and leaves its |rs|^2
    // partials.
    template <int P>
    int iterate(int slot, bool restart) {
        const double k2 = -kappa * kappa;
        int n = (int)hop_partials(g, 1), rc = LQCD_OK;
        const bool few = n <= CG_FEW;
        if (P != LQCD_F16 && few) {
            rc = hop(LQCD_ODD, w.to, w.rs, nullptr, 1.0, false, P, link, U, nullptr, CG_DIR_IN, slot, nullptr, restart);
            if (!rc) rc = hop(LQCD_EVEN, w.te, w.to, w.rs, k2, false, P, link, U, w.pap, CG_DIR_Y);
            std::swap(w.p[0], w.p[1]);
        } else {
            const double *sums = w.partial;
            if (n > CG_MANY) {
                cg_groups_k<<<CG_GROUPS, 64, 0, st>>>(w.partial, n, w.groups);
                sums = w.groups;
                n = CG_GROUPS;
            }
            const int64_t blocks = (g.vh + SUM_BLOCK - 1) / SUM_BLOCK;
            cg_direction_k<P><<<dim3((unsigned)(blocks < DIR_BLOCKS ? blocks : DIR_BLOCKS)), SUM_BLOCK, 0, st>>>(
                w.p[1], w.p[0], w.rs, w.xs, w.sc, sums, n, slot, restart, g.vh);
            std::swap(w.p[0], w.p[1]);
            rc = check_launch();
            if (!rc) rc = hop(LQCD_ODD, w.to, w.p[0], nullptr, 1.0, false, P, link, U, nullptr);
            if (!rc) rc = hop(LQCD_EVEN, w.te, w.to, w.p[0], k2, false, P, link, U, w.pap);
        }
        if (!rc) rc = hop(LQCD_ODD, w.to, w.te, nullptr, 1.0, true, P, link, U, nullptr, few ? CG_NONE : CG_PRE);
        if (!rc) rc = hop(LQCD_EVEN, w.rs, w.to, w.te, k2, true, P, link, U, w.partial, CG_UPDATE, slot);
        return rc;
    }

    dim3 grid() const { return dim3((unsigned)((g.vh + CG_BLOCK - 1) / CG_BLOCK)); }

    // the sums of n partials, and of n more (second), on the host
    template <bool RESID>
    int total(const double *partial, int n, int stride, double *host, const double *second = nullptr) {
        const int nv = second ? 2 : 1;
        cg_sum_k<RESID><<<1, SUM_BLOCK, 0, st>>>(partial, second, n, stride, w.sc, mail.get(),
                                                 mail.get() ? mail.next() : 0);
        const int rc = check_launch();
        if (rc) return rc;
        if (mail.get()) return mail.wait(host, nv);
        hipError_t e = hipMemcpyAsync(host, w.sc + CG_OUT, nv * sizeof(double), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            set_hip_error(e);
            return LQCD_EHIP;
        }
        return LQCD_OK;
    }

    // |a|^2 and |b|^2 of two FP64 half fields on the host
    int norms64(const char *a, const char *b, double host[2]) {
        const int n = (int)reduce_grid(g, 1);
        launch_reduce(g, 1, a, nullptr, LQCD_F64, w.pap, st);
        launch_reduce(g, 1, b, nullptr, LQCD_F64, w.pap + 2 * n, st);
        return total<false>(w.pap, n, 2, host, w.pap + 2 * n);
    }

    // The inner residual from the true one: rs = b - A64 x64 (FP64, rounded to
    // the inner precision) with its partials, |b - A64 x64|^2 on the host.
    template <int P>
    int true_residual(char *x64, const char *b, double *rr) {
        const double k2 = -kappa * kappa;
        int rc = hop(LQCD_ODD, w.to64, x64, nullptr, 1.0, false, LQCD_F64, link64, U64, nullptr);
        if (!rc) rc = hop(LQCD_EVEN, w.te64, w.to64, x64, k2, false, LQCD_F64, link64, U64, nullptr);
        if (!rc) rc = hop(LQCD_ODD, w.to64, w.te64, nullptr, 1.0, true, LQCD_F64, link64, U64, nullptr);
        if (!rc) rc = hop(LQCD_EVEN, w.rs, w.to64, w.te64, k2, true, LQCD_F64, link64, U64, w.pap, CG_RESID + P, 0, b);
        return rc ? rc : total<true>(w.pap, (int)hop_partials(g, 1), 1, rr);
    }

    template <int P>
    int run(char *x64, const char *b, double tol, int maxiter, int reliable_every,
            lqcd_cg_stats_t *stats) {
        stats->iterations = 0;
        stats->reliable_updates = 0;
        mail.open(st);
        double norms[2] = {0.0, 0.0};
        int rc = norms64(b, x64, norms);
        if (rc) return rc;
        const double bb = norms[0], xx = norms[1];
        if (!std::isfinite(bb)) return LQCD_ENAN;
        if (bb == 0.0) {
            // the solution of A x = 0 is x = 0
            hipError_t e = hipMemsetAsync(x64, 0, half_spinor_bytes(g, LQCD_F64), st);
            if (e != hipSuccess) {
                set_hip_error(e);
                return LQCD_EHIP;
            }
            stats->true_residual = 0.0;
            stats->iterated_residual = 0.0;
            return LQCD_OK;
        }
        const double target = tol * tol * bb;
        double rr = 0.0;
        // a zero starting guess (the common case) needs no FP64 operator
        // application: r = b
        if (xx == 0.0) rr = bb;
        else rc = true_residual<P>(x64, b, &rr);
        if (rc) return rc;
        if (!std::isfinite(rr)) return LQCD_ENAN;
        stats->true_residual = std::sqrt(rr / bb);
        stats->iterated_residual = stats->true_residual;
        if (rr <= target) return LQCD_OK;

        // inner start: rs = b - A x, xs = 0, and p = 0 with beta = alpha = 0
        // for the first direction update
        hipError_t e = hipMemsetAsync(w.sc, 0, sizeof(double) * CG_SCALARS, st);
        if (xx == 0.0) {
            cg_start_k<P><<<grid(), CG_BLOCK, 0, st>>>(w.rs, w.xs, w.p[0], b, w.partial, g.vh);
            rc = check_launch();
        } else {
            const size_t hb = half_spinor_bytes(g, P);
            if (e == hipSuccess) e = hipMemsetAsync(w.xs, 0, hb, st);
            if (e == hipSuccess) e = hipMemsetAsync(w.p[0], 0, hb, st);
        }
        if (e != hipSuccess) {
            set_hip_error(e);
            return LQCD_EHIP;
        }
        if (rc) return rc;

        int k = 0;
        bool restart = false;
        double rr_it = rr;
        double rr_ref = rr;  // true residual at the last reliable update
        const double delta = P == LQCD_F64 ? 0.0 : P == LQCD_F32 ? DELTA_F32 : DELTA_F16;
        const double drift = delta * delta;
        const double target_inner = P == LQCD_F64 ? target : INNER_MARGIN2 * target;
        const int defer = P == LQCD_F32 ? DRIFT_DEFER : 0;
        // residual at the last host read, the decay of log(rr) per iteration
        // between the last two reads (kept across reliable updates), and the
        // iteration of the next read
        int k_seen = 0;
        double rr_seen = rr;
        double rate = 0.0;
        int next_read = CHECK_EVERY;
        while (true) {
            rc = iterate<P>(k & 1, restart);
            restart = false;
            if (rc) return rc;
            ++k;
            bool reliable = reliable_every > 0 && k % reliable_every == 0;
            if (reliable || k >= next_read || k >= maxiter) {
                rc = total<false>(w.partial, (int)hop_partials(g, 1), 1, &rr_it);
                if (rc) return rc;
                if (!std::isfinite(rr_it)) {
                    stats->iterations = k;
                    return LQCD_ENAN;
                }
                if (k > k_seen && rr_it > 0.0 && rr_it < rr_seen)
                    rate = std::log(rr_it / rr_seen) / (double)(k - k_seen);
                const int left = iterations_left(rr_it, rate, target_inner);
                if (rr_it <= target_inner) reliable = true;
                if (rr_it < drift * rr_ref && (left > defer || rr_it < DRIFT_HARD * drift * rr_ref))
                    reliable = true;
                next_read = k + read_gap(left);
                rr_seen = rr_it;
                k_seen = k;
            }
            if (reliable || k >= maxiter) {
                cg_fold_k<P><<<grid(), CG_BLOCK, 0, st>>>(x64, w.xs, w.p[0], w.sc, g.vh);
                rc = true_residual<P>(x64, b, &rr);
                if (rc) return rc;
                stats->reliable_updates += 1;
                stats->iterations = k;
                stats->true_residual = std::sqrt(rr / bb);
                stats->iterated_residual = std::sqrt(rr_it / bb);
                if (!std::isfinite(rr)) return LQCD_ENAN;
                if (rr <= target) return LQCD_OK;
                if (k >= maxiter) return LQCD_ENOCONV;
                rr_ref = rr;
                // the inner residual restarts from the FP64 one
                restart = rr > RESTART * rr_it;
                rr_seen = rr;
                k_seen = k;
                next_read = k + read_gap(iterations_left(rr, rate, target_inner));
            }
        }
    }
};

}  // namespace lqcd

using namespace lqcd;

extern "C" size_t lqcd_cg_workspace_bytes(const lqcd_geom_t *gg, int inner_prec, int inner_link) {
    Geom g;
    if (!make_geom(gg, &g) || !valid_link(inner_prec, inner_link)) return 0;
    return cg_layout(g, inner_prec, nullptr).bytes;
}

extern "C" int lqcd_cg_solve(const lqcd_geom_t *gg, void *x_e, const void *b_e, const void *U_hi,
                             int link_hi, const void *U_lo, int inner_prec, int inner_link,
                             double kappa, double tol, int maxiter, int reliable_every,
                             void *workspace, size_t workspace_bytes, lqcd_cg_stats_t *stats,
                             void *stream) {
    const auto t0 = std::chrono::steady_clock::now();
    lqcd_cg_stats_t local{};
    lqcd_cg_stats_t *st = stats ? stats : &local;
    *st = lqcd_cg_stats_t{};
    Solver s{};
    auto finish = [&](int rc) {
        st->status = rc;
        st->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        return rc;
    };
    if (!make_geom(gg, &s.g)) return finish(LQCD_EINVAL);
    if (!valid_link(inner_prec, inner_link) || !valid_link(LQCD_F64, link_hi)) return finish(LQCD_EINVAL);
    if (!x_e || !b_e || !U_hi || !U_lo || !workspace) return finish(LQCD_EINVAL);
    if (((uintptr_t)x_e | (uintptr_t)b_e | (uintptr_t)U_hi | (uintptr_t)U_lo) & 15) return finish(LQCD_EINVAL);
    if ((uintptr_t)workspace & 255) return finish(LQCD_EINVAL);
    if (!(tol > 0.0) || maxiter <= 0 || reliable_every < 0 || !std::isfinite(kappa)) return finish(LQCD_EINVAL);
    if (x_e == b_e) return finish(LQCD_EINVAL);
    s.w = cg_layout(s.g, inner_prec, (char *)workspace);
    if (workspace_bytes < s.w.bytes) return finish(LQCD_ESMALL);
    s.st = (hipStream_t)stream;
    s.kappa = kappa;
    s.prec = inner_prec;
    s.link = inner_link;
    s.U = (const char *)U_lo;
    s.U64 = (const char *)U_hi;
    s.link64 = link_hi;
    int rc;
    if (inner_prec == LQCD_F64) rc = s.run<LQCD_F64>((char *)x_e, (const char *)b_e, tol, maxiter, reliable_every, st);
    else if (inner_prec == LQCD_F32) rc = s.run<LQCD_F32>((char *)x_e, (const char *)b_e, tol, maxiter, reliable_every, st);
    else rc = s.run<LQCD_F16>((char *)x_e, (const char *)b_e, tol, maxiter, reliable_every, st);
    // (a solve that failed may have failed because its stream is captured,
    // where an event would become part of the graph)
    const hipError_t e = rc == LQCD_OK ? drain_stream(s.st) : hipStreamSynchronize(s.st);
    if (e != hipSuccess && rc == LQCD_OK) {
        set_hip_error(e);
        rc = LQCD_EHIP;
    }
    return finish(rc);
}
