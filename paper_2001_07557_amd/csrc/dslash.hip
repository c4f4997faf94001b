// Wilson hopping term on gfx950: one thread per output site, eight
// neighbour hops with spin projection to half-spinors, SU(3) x half-spinor
// products and reconstruction into the four spin rows, boundary signs applied
// in the kernel, fused alpha*D + beta*y epilogue and an optional fused |out|^2
// block partial for the solver.
//
// The operator is the one the paper benchmarks in Sec. 3.3 (Fig. 4d); its
// definition (hopping form, DeGrand-Rossi basis) is spelled out in lqcd.h.
// The paper's kernels vectorise over sites packed into long vector registers
// (Sec. 3.1) and need lane permutations at sublattice boundaries; here each
// lane owns one site and neighbours are plain indexed loads, so no lane
// permutation exists.

#include <type_traits>

#include "lqcd_internal.h"
#include "reduce.h"
#include "hop_common.h"

namespace lqcd {

// Cache hints of the hop kernels:
//  * output stores are non-temporal: the output is not read again by the same
//    launch, and a later launch reads it on other XCDs, whose L2s do not
//    share it, so keeping it in this XCD's L2 only evicts the neighbour
//    spinors held there for reuse;
//  * link loads are non-temporal when the links plus the input spinor exceed
//    the 256 MB Infinity Cache in front of HBM; when they fit, plain loads
//    leave them cached for the next application.  A launch over both
//    parities uses every link twice and always loads them plainly (48^3x96
//    full-lattice M, FP32-18: 4.4 -> 5.1 TB/s).
// Measured (fraction of 8 TB/s, alternating D_eo / D_oe): streaming the
// output takes FP64-18 from 67.0 to 78.3 at 32^4 and from 64.0 to 68.6 at
// 48^3x96; cached rather than streamed links take FP32-12 from 75.4 to 83.9
// at 32^4 (201 MB of links) and FP64-18 from 56.6 to 66.7 at 16^4.  The same
// hint on the spinor loads would destroy the L2 reuse (LQCD_SPINOR_NT,
// FP64-18 at 32^4: 51%).  LQCD_OUT_NT / LQCD_LINK_NT = 0 switch a hint off,
// LQCD_HOP_STREAM = 0..3 forces the mode (ablations).
#ifndef LQCD_HOP_STREAM
#define LQCD_HOP_STREAM -1
#endif
// row-parallel rebuild of the FP32 hop on small lattices (ablation switch)
#ifndef LQCD_HOP_ROWS
#define LQCD_HOP_ROWS 1
#endif
// both-parity launches pair the even and odd tile of a region (ablation switch)
#ifndef LQCD_HOP_ARGS_TOUCH
#define LQCD_HOP_ARGS_TOUCH 1
#endif
#ifndef LQCD_HOP_PAIRED
#define LQCD_HOP_PAIRED 1
#endif
// Blocks in flight of the FP64 4-way kernel.  By its 36 KB of LDS four blocks
// fit a CU, and by registers where an instance has at most 128 VGPRs: 114-120
// without a y term and on small lattices, 126 for the large adjoint with one;
// the large forward ones that read y early have 130-132, a canonical FP64
// result 132, the CG update 148, and fit three whatever the LDS.  With four an
// XCD's 32 CUs keep 128 tiles in flight, more than one t-slice of its z-slab:
// the three input t-slices the brick order relies on no longer fit its 4 MB L2
// beside them.  Even-odd launches from V/2 >= 2^17 and both-parity launches
// from 2^15 add dynamic LDS that leaves three blocks per CU.  Measured (us, four
// -> three -> two blocks per CU, y read late, 120 VGPRs): full-lattice M 24^4
// FP64-18 81.4 -> 78.5 -> 80.6, FP64-12 67.8 -> 67.1 -> 71.2; 32^4 FP64-18 238.5 -> 228.7 -> 236.5, FP64-12 196.2 -> 193.4 ->
// 209.5; 48^3x96 FP64-18 2470 -> 2397 -> 2445, FP64-12 2016 -> 1996 -> 2156;
// 16^3x32 FP64-18 33.8 -> 32.6; Mhat 32^4 FP64-18 285.1 -> 283.7, 28^4
// FP64-18 175.6 -> 173.5, 38^3x40 FP64-12 -> 512 -> 527, 48^3x96 FP64-12
// -> 2489 -> 2526, but 16^3x32 FP64-12 27.7 -> 29.4 (below the line).  The
// launches that want two blocks are both-parity 18-real ones in plain order
// (38^2x14x40 -> 214 -> 210) or in slab order where the three t-slices of both
// halves (144 bytes per site of a t-slice and slab) overflow the L2: 38^3x40
// 575 -> 536 -> 522, 46^3x50 1318 -> 1221 -> 1180; at 28^4 (1.6 MB) three are
// ahead, 147.0 -> 140.5 -> 144.4.
// With y read early the limit acts on the adjoint, the small instances and the
// launches that want two: M^dag FP64-18 32^4 236.6 -> 226.9 us and 1433 -> 1256
// MB fetched, 28^4 146.9 -> 140.1 and 923 -> 841, 38^3x40 (two) 579.7 -> 507.1
// and 4151 -> 3333; the large forward M has the same times and bytes without it.
// binary16 storage (also 4-way) loses 8 points with two and keeps what fits.
// LQCD_HOP_EXTRA_LDS forces a value for every 4-way launch (ablations).
constexpr uint32_t F64_LDS_THREE = 6144, F64_LDS_TWO = 18432;
constexpr int64_t F64_SLAB_TWO_BYTES = (int64_t)3 << 20;
#ifndef LQCD_HOP_F64_LDS_MIN_LOG2
#define LQCD_HOP_F64_LDS_MIN_LOG2 17
#endif
// (t-region launches, short as they are, only from 2^20: 32^3x8 FP64-18 face
// pack, interior and boundary 49.6 us with three blocks, 48.9 with four; the
// forward ones with streamed links and a y term fit three by their registers)
#ifndef LQCD_HOP_F64_REGION_LDS_MIN_LOG2
#define LQCD_HOP_F64_REGION_LDS_MIN_LOG2 20
#endif
#ifndef LQCD_HOP_F64_PAIRED_LDS_MIN_LOG2
#define LQCD_HOP_F64_PAIRED_LDS_MIN_LOG2 15
#endif
#ifndef LQCD_HOP_EXTRA_LDS
#define LQCD_HOP_EXTRA_LDS -1
#endif
// t-march form of the 4-way shape: t-slices per block (0 = off), used from
// V/2 >= 2^LQCD_HOP_TMARCH_MIN_LOG2 sites
#ifndef LQCD_HOP_TMARCH
#define LQCD_HOP_TMARCH 0
#endif
#ifndef LQCD_HOP_TMARCH_MIN_LOG2
#define LQCD_HOP_TMARCH_MIN_LOG2 17
#endif
// Whole-lattice even-odd launches with odd output (V/2 >= 2^17) walk every
// XCD's range of tiles backwards.  Operators alternate output parities (Mhat, its adjoint,
// the solver's four hops), and a hop that starts where the one before it
// ended finds the last links and spinors of that one in the Infinity Cache;
// walked the same way round, a working set beyond 256 MB has evicted what the
// next launch reads first.  Mhat, three field sets in turn (us, same way ->
// back and forth, two runs each): 32^4 FP32-12 113.0-113.5 -> 108.5, FP64-12
// 227.9-228.7 -> 226.6, FP64-18 285.4 -> 284.8; 48^3x96 FP32-12 1172 -> 1151,
// 48^4 FP64-18 1583 -> 1562.  Loading the links of the last 48-200 MB of a
// launch plainly, to keep more of them, gained another 1-3% at 24^3x48 and
// lost 1.5% at 48^3x96 (twice the code), so the link hint stays per launch.
// 0 switches it off (ablation).
#ifndef LQCD_HOP_ZIGZAG
#define LQCD_HOP_ZIGZAG 1
#endif
constexpr int64_t INFINITY_CACHE_BYTES = (int64_t)256 << 20;

template <int P>
__device__ __forceinline__ void cg_new_p(const HopArgs &a, int p, int64_t s,
                                         cplx<typename real_of<P>::type> v[12]);

// What the epilogue of a site adds (DIR: y is the new direction).  Launches
// whose links are streamed (NTM bit 1: even-odd, beyond the Infinity Cache),
// FP64 and FP32, read it before the barrier that the epilogue waits at, so that
// its latency passes meanwhile: Mhat 32^4 FP64-18 281.4 -> 278.7 us, 48^3x96
// FP32-12 1163 -> 1154.  The others read it after: small launches lose by it
// (Mhat 16^4 FP32-12 10.60 -> 10.76 us, also with a switch at run time),
// binary16 ones too (32^4 solve 9.29 -> 9.37 ms), and CG_UPDATE needs the
// registers (24^3x48 FP32 solve 8.23 -> 8.25 ms).
template <int P, int NORM, int NTM>
constexpr bool early_y() { return (NTM & 2) != 0 && P != LQCD_F16 && NORM != 2; }
template <int P, bool HASY, bool DIR>
__device__ __forceinline__ void load_y(const HopArgs &a, int p, int64_t s,
                                       cplx<typename real_of<P>::type> y[12]) {
    if constexpr (DIR) cg_new_p<P>(a, p, s, y);
    else if constexpr (HASY) load_spinor<P>(a.y[p], s, y);
}

// acc = alpha acc + beta y.  The fused product is spelled out, so that every
// instance rounds alike (the compiler may fuse either one).
template <int P, bool HASY>
__device__ __forceinline__ void hop_combine(const HopArgs &a, const cplx<typename real_of<P>::type> y[12],
                                            cplx<typename real_of<P>::type> acc[12]) {
    using T = typename real_of<P>::type;
    const T alpha = (T)a.alpha;
    if constexpr (HASY) {
        const T beta = (T)a.beta;
#pragma unroll
        for (int k = 0; k < 12; ++k)
            acc[k] = {fmad(alpha, acc[k].re, beta * y[k].re), fmad(alpha, acc[k].im, beta * y[k].im)};
    } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = scale(alpha, acc[k]);
    }
}

// Epilogue shared by the kernel shapes: out = alpha acc + beta y; NORM = 1
// also returns |out|^2 of the site; NORM = 2 (CG_UPDATE, with a y term) stores
// nothing of out = A p but updates r -= cg_alpha A p in place (r at a.out) and
// returns |r|^2 of the site.  x += alpha p waits for the pass that reads p
// next anyway (the direction update): one vector less per iteration, and
// fewer registers here.
template <int P, bool HASY, int NORM, bool NT>
__device__ __forceinline__ double hop_epilogue(const HopArgs &a, int p, int64_t s,
                                               const cplx<typename real_of<P>::type> y[12],
                                               cplx<typename real_of<P>::type> acc[12],
                                               double cg_alpha = 0.0) {
    using T = typename real_of<P>::type;
    hop_combine<P, HASY>(a, y, acc);
    if constexpr (NORM == 2) {
        const T c = (T)cg_alpha;
        cplx<T> vr[12];
        load_spinor<P>(a.out[p], s, vr);
        T nr = 0;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            vr[k] = {vr[k].re - c * acc[k].re, vr[k].im - c * acc[k].im};
            nr += norm2(vr[k]);
        }
        store_spinor<P>(a.out[p], s, vr);
        return (double)nr;
    }
    double nrm = 0.0;
    if constexpr (NORM == 1) {
        T t = 0;
#pragma unroll
        for (int k = 0; k < 12; ++k) t += norm2(acc[k]);
        nrm = (double)t;
    }
    store_spinor<P, NT>(a.out[p], s, acc);
    return nrm;
}

// CG_RESID: r = rhs - (alpha acc + y) of the site, stored in precision PI;
// nrm = |r|^2 in FP64 and |r as stored|^2.
template <int P, int PI>
__device__ __forceinline__ void cg_residual(const HopArgs &a, int p, int64_t s,
                                            const cplx<typename real_of<P>::type> y[12],
                                            cplx<typename real_of<P>::type> acc[12], double nrm[2]) {
    using TI = typename real_of<PI>::type;
    hop_combine<P, true>(a, y, acc);
    cplx<double> b[12];
    cplx<TI> r[12];
    load_spinor<LQCD_F64>(a.rhs, s, b);
    double n = 0.0;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        b[k] = {b[k].re - acc[k].re, b[k].im - acc[k].im};
        n += norm2(b[k]);
        r[k] = {(TI)b[k].re, (TI)b[k].im};
    }
    nrm[0] = n;
    nrm[1] = (double)store_spinor<PI>(a.out[p], s, r, true);
}

// CG_DIR_Y, wave 1: x += alpha p old of the site; wave 2: the new p.  Both
// wait for nothing that wave 0 does.
template <int P>
__device__ __forceinline__ void cg_step_x(const HopArgs &a, int64_t s) {
    using T = typename real_of<P>::type;
    const T c = (T)a.sc[CG_ALPHA];
    cplx<T> vp[12], vx[12];
    load_spinor<P>(a.p_old, s, vp);
    load_spinor<P>(a.x, s, vx);
#pragma unroll
    for (int k = 0; k < 12; ++k) vx[k] = {fmad(c, vp[k].re, vx[k].re), fmad(c, vp[k].im, vx[k].im)};
    store_spinor<P>(a.x, s, vx);
}
template <int P>
__device__ __forceinline__ void cg_new_p(const HopArgs &a, int p, int64_t s,
                                         cplx<typename real_of<P>::type> v[12]) {
    using T = typename real_of<P>::type;
    const T b = (T)a.sc[CG_BETA];
    cplx<T> vp[12];
    load_spinor<P>(a.y[p], s, v);  // r
    load_spinor<P>(a.p_old, s, vp);
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = {fmad(b, vp[k].re, v[k].re), fmad(b, vp[k].im, v[k].im)};
}

// CG_UPDATE: alpha of this iteration, formed by one wave; block 0 keeps it.
__device__ __forceinline__ double cg_alpha_of(const HopArgs &a) {
    const double pap = wave_total(a.sums, a.n_sums);
    // <p, A p> = 0 only when p = 0: the iteration has terminated exactly
    // (e.g. a source spanned by few eigenvectors); take no step and let the
    // next residual check confirm convergence.
    const double alpha = pap > 0.0 ? a.sc[CG_RR + a.slot] / pap : 0.0;
    if (blockIdx.x == 0 && (threadIdx.x & 63) == 0) a.sc[CG_ALPHA] = alpha;
    return alpha;
}

// CG_PRE: this block's run of the partials, summed by one wave.
__device__ __forceinline__ void cg_presum(const HopArgs &a) {
    if (blockIdx.x >= (uint32_t)a.n_groups) return;
    const int per = (a.n_sums + a.n_groups - 1) / a.n_groups;
    const int lo = (int)blockIdx.x * per;
    const int n = a.n_sums - lo < per ? a.n_sums - lo : per;
    const double t = wave_total(a.sums + lo, n);
    if ((threadIdx.x & 63) == 0) a.groups[blockIdx.x] = t;
}

// Canonical output (CT: its real type): wave 0 stages the tile's sites in LDS
// the staging of the hops no longer needs, and the whole block writes them.
// Every thread of the block calls it.  The extra barrier and LDS pass cost 8 us
// of an 88 us launch (24^4, FP64) and save the 24 us (and 130 MB) of a
// separate unpacking pass.
template <typename CT, int P, bool HASY, int THREADS>
__device__ __forceinline__ void hop_canon(const HopArgs &a, int p, int64_t s, bool mine,
                                          const cplx<typename real_of<P>::type> y[12],
                                          cplx<typename real_of<P>::type> acc[12], v4u *stage) {
    constexpr int GS = spinor_granules<CT>();
    const int lane = threadIdx.x & 63;
    if (mine) {
        hop_combine<P, HASY>(a, y, acc);
        // the reads of the staged hops come before these writes of another type
        asm volatile("" ::: "memory");
        CT *d = reinterpret_cast<CT *>(stage + lane * (GS + 1));
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            d[2 * k] = (CT)acc[k].re;
            d[2 * k + 1] = (CT)acc[k].im;
        }
    }
    __syncthreads();
    canon_store<GS, THREADS>(a.g, reinterpret_cast<v4u *>(a.out[0]), p, s - lane, stage);
}

// The five fields read first lie on the five 64-byte lines of the arguments.
static_assert(offsetof(HopArgs, sc) <= 5 * 64 && sizeof(HopArgs) <= 7 * 64,
              "the fields read first span five lines, the solver's the ones after them");
static_assert(offsetof(HopArgs, bpp) / 64 == 0 &&
                  (offsetof(HopArgs, g) + offsetof(Geom, lxh)) / 64 == 1 &&
                  (offsetof(HopArgs, g) + offsetof(Geom, vh)) / 64 == 2 &&
                  offsetof(HopArgs, in) / 64 == 3 && offsetof(HopArgs, stream) / 64 == 4,
              "one touched field per line of the launch arguments");

// Output parity and checkerboard site of this thread (block = one 64-site
// tile).  A launch over both parities gives consecutive blocks the even and
// the odd tile of one region: each reads the links and spinors of the other,
// so both are fetched into the same XCD's L2 once.
// BIG (V/2 >= 2^BIG_MIN_LOG2): the launch may walk backwards or in slab order.
// On smaller lattices, whose launches are as long as the chain from the
// arguments to the first load, the few scalar instructions of either cost
// 0.07 us of 3.95 (16^4 FP32-12; 0.1-0.2 of 3.73 binary16), so their kernels
// are instances of their own.
constexpr int BIG_MIN_LOG2 = LQCD_BRICK_MIN_LOG2;
template <bool BIG>
__device__ __forceinline__ int64_t hop_site_index(const HopArgs &a, int lane, int &p, int64_t &blk) {
    // selects, not branches: every launch argument is read up front
#if LQCD_HOP_ARGS_TOUCH
    // one field from each 64-byte line of the arguments, needed before
    // anything else: the lines come in with one scalar-cache miss instead of
    // one after each dependent step
    asm volatile("" ::"s"(a.bpp), "s"(a.g.lxh), "s"(a.g.vh), "s"(a.in[0]), "s"(a.stream));
#endif
    const uint32_t bx = blockIdx.x;
    blk = LQCD_HOP_XCD ? xcd_block(bx, a.nblk, BIG ? a.rev : 0) : (int64_t)bx;
    // paired: blocks 2i / 2i + 1 take the even / odd tile i; otherwise the
    // first bpp blocks take parity par0 and the rest the other parity
    const int q = blk >= a.bpp ? 1 : 0;
    const uint32_t lb = (uint32_t)(a.paired ? blk >> 1 : blk - q * a.bpp);
    p = a.paired ? (int)(blk & 1) : a.par0 ^ q;
    const int64_t tile = brick_order<BIG>(lb, a.brick, a.g);
    // the partial of a tile in slab order, whose blocks outnumber the tiles,
    // goes by the tile
    if (BIG && a.brick.lz == 0) blk = tile;
    return tile * HOP_SITES + lane;
}

// 4-way shape: wave w computes both hops of direction w; waves 1..3 leave
// their partial spinors in LDS and wave 0 adds them up.  CT: real type of a
// canonical output, void for the internal layout.
template <int P, int LK, bool DAG, bool HASY, int NORM, int NTM, bool HALO, typename CT = void, int CG = CG_NONE,
          bool BIG = true>
__global__ __launch_bounds__(256) void hop4_kernel(HopArgs a) {
    using T = typename real_of<P>::type;
    __shared__ alignas(16) cplx<T> part[3][12][64];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    int p;
    int64_t blk;
    const int64_t s = hop_site_index<BIG>(a, lane, p, blk);
    const Geom &g = a.g;
    const bool active = s < g.vh;
    // (coordinates of a padding site are never used, and s < 2^31 anyway;
    // CG_DIR_IN sums with whole waves, whose lanes past the last site repeat
    // its hops)
    const int64_t sl = CG == CG_DIR_IN && !active ? g.vh - 1 : s;
    const Coord c = cb_coords(g, p, sl);
    cplx<T> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = {0, 0};
    DirIn<T> dir{&a, 0};
    DirIn<T> *const d = CG == CG_DIR_IN ? &dir : nullptr;
    if (active || CG == CG_DIR_IN) {
        constexpr bool LNT = (NTM & 2) != 0;
        switch (w) {
            case 0: hop_direction<0, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, acc, nullptr, d); break;
            case 1: hop_direction<1, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, acc, nullptr, d); break;
            case 2: hop_direction<2, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, acc, nullptr, d); break;
            default: hop_direction<3, P, LK, DAG, LNT, HALO>(g, a.in[p], a.U, p, sl, c, acc, a.face, d); break;
        }
    }
    if (w > 0) {
#pragma unroll
        for (int k = 0; k < 12; ++k) part[w - 1][k][lane] = acc[k];
    }
    __shared__ double alpha;
    if (NORM == 2 && w == 1) {
        const double t = cg_alpha_of(a);
        if (lane == 0) alpha = t;
    }
    if constexpr (CG == CG_DIR_Y) {
        if (w == 1 && active) cg_step_x<P>(a, s);
        if (w == 2 && active) {
            cplx<T> v[12];
            cg_new_p<P>(a, p, s, v);
            store_spinor<P>(a.p_new, s, v);
        }
    }
    if (CG == CG_PRE && w == 3) cg_presum(a);
    cplx<T> y[12];
    constexpr bool early = early_y<P, NORM, NTM>();
    if (early && w == 0 && active) load_y<P, HASY, CG == CG_DIR_Y>(a, p, s, y);
    __syncthreads();
    // (FP64 on large lattices: before the LDS sums, M 32^4 FP64-12 193.4 -> 191.3
    // us; on small ones after them, where neither order was measurably faster:
    // Mhat 20^3x18 FP64-18 47.7 to 47.9)
    constexpr bool first_y = P == LQCD_F64 && CG != CG_DIR_Y && BIG;
    double nrm[2] = {0.0, 0.0};
    if (w == 0 && active) {
        if (!early && first_y) load_y<P, HASY, CG == CG_DIR_Y>(a, p, s, y);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = acc[k] + part[j][k][lane];
        if (!early && !first_y) load_y<P, HASY, CG == CG_DIR_Y>(a, p, s, y);
        if constexpr (CG >= CG_RESID)
            cg_residual<P, CG - CG_RESID>(a, p, s, y, acc, nrm);
        else if constexpr (std::is_void<CT>::value)
            nrm[0] = hop_epilogue<P, HASY, NORM, (NTM & 1) != 0>(a, p, s, y, acc, NORM == 2 ? alpha : 0.0);
    }
    if constexpr (!std::is_void<CT>::value) {
        static_assert(canon_stage_bytes<spinor_granules<CT>()>() <= sizeof(part), "the tile fits the staging");
        hop_canon<CT, P, HASY, 256>(a, p, s, w == 0 && active, y, acc, reinterpret_cast<v4u *>(part));
    }
    if constexpr (NORM) {
        // wave 0 holds every site of the tile: a wave reduction suffices and
        // the other waves leave after the staging barrier
        if (w == 0) {
            const double t = wave_sum(nrm[0]);
            if (lane == 0 && blk < a.g.ntiles) a.partial[blk] = t;
            if constexpr (CG >= CG_RESID) {
                const double u = wave_sum(nrm[1]);
                if (lane == 0 && blk < a.g.ntiles) a.stored[blk] = u;
            }
        }
    }
}

// t-march form of the 4-way shape (LQCD_HOP_TMARCH = t-slices per block):
// a block walks one tile column, the same 64 in-slice sites of tseg
// consecutive t-slices.  The t-neighbours of a tile are the same lanes of
// the tiles one slice up and one down, so the wave of direction t loads each
// input t-slice of its column once: the load of input slice t + 1 gives the
// forward hop of output slice t and the backward hop of output slice t + 2,
// whose two colour vectors wait two steps in a lane-private LDS ring (the
// 4-way form loads that input again two output slices later, from the L2
// if it is still there).  Waves 0-2 read their neighbours as in the 4-way
// shape; XCD x of 8 takes columns [x K/8, (x + 1) K/8) of every segment, so
// the blocks of one XCD walk its z-slab side by side.  Same arithmetic, in
// the same order, as the 4-way shape: the results are bit-identical.
template <int P, int LK, bool DAG, bool HASY, int NORM, int NTM>
__global__ __launch_bounds__(256) void hop4t_kernel(HopArgs a) {
    using T = typename real_of<P>::type;
    using E = typename hop_elem<P>::type;
    using PR = Proj<3>;
    constexpr bool LNT = (NTM & 2) != 0;
    constexpr int SF = DAG ? 1 : -1;
    constexpr int SB = -SF;
    constexpr int r0 = SF > 0 ? conj_code(PR::c0) : neg_code(conj_code(PR::c0));
    constexpr int r1 = SF > 0 ? conj_code(PR::c1) : neg_code(conj_code(PR::c1));
    __shared__ cplx<T> part[3][12][64];
    __shared__ cplx<T> ring[2][6][64];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const Geom &g = a.g;
    const int p = a.par0;
    const int lt = g.L[3];
    const uint32_t kx = (uint32_t)(g.st >> TILE_SHIFT) / 8;  // columns per XCD
    const uint32_t b = blockIdx.x;
    const uint32_t j = b >> 3;
    const uint32_t seg = j / kx;
    const uint32_t col = (b & 7) * kx + (j - seg * kx);
    const int t0 = (int)seg * a.tseg;
    const int t1 = t0 + a.tseg < lt ? t0 + a.tseg : lt;
    const int64_t s0 = (int64_t)col * TILE + lane;  // this lane's site of slice 0
    const char *in = a.in[p];
    // backward t-hop of output slice t from input slice t - 1 (wrapping, with
    // the boundary sign), as the 4-way shape forms it
    auto bwd_half = [&](int t, cplx<T> bh[6]) {
        const bool wrap = t == 0;
        const int64_t nb = (int64_t)(wrap ? lt - 1 : t - 1) * g.st + s0;
        T sgn = wrap && g.bc[3] < 0 ? T(-1) : T(1);
        cplx<E> psi[12];
        load_spinor_hop<P>(in, nb, psi, sgn);
        link_chi<3, SB, true, P, LK, LNT>(a.U, g.ntiles, p ^ 1, nb, psi, sgn, bh, bh + 3);
    };
    if (w == 3) {
        for (int t = t0; t < t0 + 2 && t < t1; ++t) {
            cplx<T> bh[6];
            bwd_half(t, bh);
#pragma unroll
            for (int k = 0; k < 6; ++k) ring[t & 1][k][lane] = bh[k];
        }
    }
    for (int t = t0; t < t1; ++t) {
        const int64_t s = (int64_t)t * g.st + s0;
        const Coord c = cb_coords(g, p, s);
        cplx<T> acc[12];
        switch (w) {
            case 0: hop_direction<0, P, LK, DAG, LNT>(g, in, a.U, p, s, c, acc); break;
            case 1: hop_direction<1, P, LK, DAG, LNT>(g, in, a.U, p, s, c, acc); break;
            case 2: hop_direction<2, P, LK, DAG, LNT>(g, in, a.U, p, s, c, acc); break;
            default: {
                // forward hop: input slice t + 1 (wrapping), link U_t(s)
                const bool wrap = t == lt - 1;
                const int64_t nb = (int64_t)(wrap ? 0 : t + 1) * g.st + s0;
                T sgn = wrap && g.bc[3] < 0 ? T(-1) : T(1);
                cplx<E> psi[12];
                cplx<T> f[6];
                load_spinor_hop<P>(in, nb, psi, sgn);
                link_chi<3, SF, false, P, LK, LNT>(a.U, g.ntiles, p, s, psi, sgn, f, f + 3);
                hop_fence<T, 6>(f);
                cplx<T> bh[6];
#pragma unroll
                for (int k = 0; k < 6; ++k) bh[k] = ring[t & 1][k][lane];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    acc[q] = f[q] + bh[q];
                    acc[3 + q] = f[3 + q] + bh[3 + q];
                    acc[PR::a0 * 3 + q] = mul_unit<r0>(f[q] - bh[q]);
                    acc[PR::a1 * 3 + q] = mul_unit<r1>(f[3 + q] - bh[3 + q]);
                }
                hop_fence<T, 12>(acc);
                // the same input gives the backward hop of output slice t + 2
                // (never across the boundary inside a segment, so the sign
                // factor is the forward hop's: 1, times the binary16 scale)
                if (t + 2 < t1) {
                    link_chi<3, SB, true, P, LK, LNT>(a.U, g.ntiles, p ^ 1, nb, psi, sgn, bh, bh + 3);
#pragma unroll
                    for (int k = 0; k < 6; ++k) ring[t & 1][k][lane] = bh[k];
                }
            }
        }
        __syncthreads();  // wave 0 has read the partials of the step before
        if (w > 0) {
#pragma unroll
            for (int k = 0; k < 12; ++k) part[w - 1][k][lane] = acc[k];
        }
        __syncthreads();
        if (w == 0) {
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < 12; ++k) acc[k] = acc[k] + part[q][k][lane];
            cplx<T> y[12];
            load_y<P, HASY, false>(a, p, s, y);
            const double nrm = hop_epilogue<P, HASY, NORM, (NTM & 1) != 0>(a, p, s, y, acc,
                                                                           NORM == 2 ? cg_alpha_of(a) : 0.0);
            if constexpr (NORM != 0) {
                const double tot = wave_sum(nrm);
                if (lane == 0) a.partial[s >> TILE_SHIFT] = tot;
            }
        }
    }
}

// 1-way shape (ablation builds, LQCD_HOP_SHAPE_* = 1): one wave per block,
// every thread computes all eight hops of its site in registers, no LDS.
// The four directions are added in the 4-way shape's order.
template <int P, int LK, bool DAG, bool HASY, int NORM, int NTM, bool HALO>
__global__ __launch_bounds__(64) void hop1_kernel(HopArgs a) {
    using T = typename real_of<P>::type;
    const int lane = threadIdx.x & 63;
    int p;
    int64_t blk;
    const int64_t s = hop_site_index<true>(a, lane, p, blk);
    const Geom &g = a.g;
    const bool active = s < g.vh;
    const Coord c = cb_coords(g, p, s);
    cplx<T> acc[12], d[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = {0, 0};
    double nrm[1] = {0.0};
    double alpha = 0.0;
    if constexpr (NORM == 2) alpha = cg_alpha_of(a);  // (a sum over the whole wave)
    if (active) {
        constexpr bool LNT = (NTM & 2) != 0;
        hop_direction<0, P, LK, DAG, LNT>(g, a.in[p], a.U, p, s, c, acc);
        hop_direction<1, P, LK, DAG, LNT>(g, a.in[p], a.U, p, s, c, d);
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = acc[k] + d[k];
        hop_direction<2, P, LK, DAG, LNT>(g, a.in[p], a.U, p, s, c, d);
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = acc[k] + d[k];
        hop_direction<3, P, LK, DAG, LNT, HALO>(g, a.in[p], a.U, p, s, c, d, a.face);
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = acc[k] + d[k];
        load_y<P, HASY, false>(a, p, s, d);
        nrm[0] = hop_epilogue<P, HASY, NORM, (NTM & 1) != 0>(a, p, s, d, acc, alpha);
    }
    if constexpr (NORM) {
        const double t = wave_sum(nrm[0]);
        if (lane == 0 && blk < a.g.ntiles) a.partial[blk] = t;
    }
}

template <int H, int P, bool DAG>
__device__ __forceinline__ void add_staged(const cplx<typename real_of<P>::type> (*chi)[6][64],
                                           int lane, cplx<typename real_of<P>::type> acc[12]) {
    using T = typename real_of<P>::type;
    cplx<T> x0[3], x1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        x0[a] = chi[H][a][lane];
        x1[a] = chi[H][3 + a][lane];
    }
    chi_accumulate<H / 2, HopSign<H, DAG>::value>(x0, x1, acc);
}

// Spin row R of the output from the eight staged half-spinors: every hop
// adds its chi0 to row 0, its chi1 to row 1 and a unit times one of them to
// row a0 or a1 of its direction.
template <int R, int H, int P, bool DAG>
__device__ __forceinline__ void row_staged(const cplx<typename real_of<P>::type> (*chi)[6][64],
                                           int lane, cplx<typename real_of<P>::type> row[3]) {
    using PR = Proj<H / 2>;
    constexpr int S = HopSign<H, DAG>::value;
    constexpr int r0 = S > 0 ? conj_code(PR::c0) : neg_code(conj_code(PR::c0));
    constexpr int r1 = S > 0 ? conj_code(PR::c1) : neg_code(conj_code(PR::c1));
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if constexpr (R == 0) row[a] = row[a] + chi[H][a][lane];
        else if constexpr (R == 1) row[a] = row[a] + chi[H][3 + a][lane];
        else if constexpr (R == PR::a0) row[a] = row[a] + mul_unit<r0>(chi[H][a][lane]);
        else row[a] = row[a] + mul_unit<r1>(chi[H][3 + a][lane]);
    }
}

// Row-parallel rebuild (FP32 storage, out = alpha D in): wave R builds and
// stores spin row R, i.e. complexes 3R .. 3R + 2 of the site, which straddle
// the 16-byte words of the tile, so they are stored as three 8-byte halves.
template <int R, int P, bool DAG, bool NT>
__device__ __forceinline__ void rebuild_row(const HopArgs &a, int p, int64_t s,
                                            const cplx<typename real_of<P>::type> (*chi)[6][64],
                                            int lane) {
    static_assert(P == LQCD_F32, "row stores assume the FP32 tile layout");
    using T = typename real_of<P>::type;
    cplx<T> row[3] = {{0, 0}, {0, 0}, {0, 0}};
    row_staged<R, 0, P, DAG>(chi, lane, row);
    row_staged<R, 1, P, DAG>(chi, lane, row);
    row_staged<R, 2, P, DAG>(chi, lane, row);
    row_staged<R, 3, P, DAG>(chi, lane, row);
    row_staged<R, 4, P, DAG>(chi, lane, row);
    row_staged<R, 5, P, DAG>(chi, lane, row);
    row_staged<R, 6, P, DAG>(chi, lane, row);
    row_staged<R, 7, P, DAG>(chi, lane, row);
    const T alpha = (T)a.alpha;
    char *t = a.out[p] + (s >> TILE_SHIFT) * spinor_tile_bytes(P) + (s & (TILE - 1)) * WORD;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int c = 3 * R + k;
        v2f *d = reinterpret_cast<v2f *>(t + (c / 2) * TILE * WORD + (c % 2) * 8);
        put<NT>(d, v2f{alpha * row[k].re, alpha * row[k].im});
    }
}

// 8-way shape: wave w computes hop w (direction w/2, forward for even w) and
// stages the two colour vectors of its multiplied half-spinor in LDS; wave 0
// rebuilds the four spin rows from the eight staged half-spinors.
template <int P, int LK, bool DAG, bool HASY, int NORM, int NTM, bool ROWS, bool HALO, typename CT = void,
          int CG = CG_NONE, bool BIG = true>
__global__ __launch_bounds__(512) void hop8_kernel(HopArgs a) {
    using T = typename real_of<P>::type;
    __shared__ alignas(16) cplx<T> chi[8][6][64];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    int p;
    int64_t blk;
    const int64_t s = hop_site_index<BIG>(a, lane, p, blk);
    const Geom &g = a.g;
    const bool active = s < g.vh;
    // (as in the 4-way shape)
    const int64_t sl = CG == CG_DIR_IN && !active ? g.vh - 1 : s;
    const Coord c = cb_coords(g, p, sl);
    DirIn<T> dir{&a, 0};
    DirIn<T> *const d = CG == CG_DIR_IN ? &dir : nullptr;
    if (active || CG == CG_DIR_IN) {
        cplx<T> x0[3], x1[3];
        constexpr bool LNT = (NTM & 2) != 0;
        switch (w) {
            case 0: hop_single<0, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, x0, x1, nullptr, d); break;
            case 1: hop_single<1, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, x0, x1, nullptr, d); break;
            case 2: hop_single<2, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, x0, x1, nullptr, d); break;
            case 3: hop_single<3, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, x0, x1, nullptr, d); break;
            case 4: hop_single<4, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, x0, x1, nullptr, d); break;
            case 5: hop_single<5, P, LK, DAG, LNT>(g, a.in[p], a.U, p, sl, c, x0, x1, nullptr, d); break;
            case 6: hop_single<6, P, LK, DAG, LNT, HALO>(g, a.in[p], a.U, p, sl, c, x0, x1, a.face, d); break;
            default: hop_single<7, P, LK, DAG, LNT, HALO>(g, a.in[p], a.U, p, sl, c, x0, x1, a.face, d); break;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            chi[w][k][lane] = x0[k];
            chi[w][3 + k][lane] = x1[k];
        }
    }
    __shared__ double alpha;
    if (NORM == 2 && w == 1) {
        const double t = cg_alpha_of(a);
        if (lane == 0) alpha = t;
    }
    if constexpr (CG == CG_DIR_Y) {
        if (w == 1 && active) cg_step_x<P>(a, s);
        if (w == 2 && active) {
            cplx<T> v[12];
            cg_new_p<P>(a, p, s, v);
            store_spinor<P>(a.p_new, s, v);
        }
    }
    if (CG == CG_PRE && w == 7) cg_presum(a);
    cplx<T> y[12];
    constexpr bool early = early_y<P, NORM, NTM>();
    if (early && w == 0 && active) load_y<P, HASY, CG == CG_DIR_Y>(a, p, s, y);
    __syncthreads();
    if constexpr (ROWS) {
        static_assert(!HASY && !NORM, "the row-parallel rebuild has no y term and no norm");
        if (active) {
            switch (w) {
                case 0: rebuild_row<0, P, DAG, (NTM & 1) != 0>(a, p, s, chi, lane); break;
                case 1: rebuild_row<1, P, DAG, (NTM & 1) != 0>(a, p, s, chi, lane); break;
                case 2: rebuild_row<2, P, DAG, (NTM & 1) != 0>(a, p, s, chi, lane); break;
                case 3: rebuild_row<3, P, DAG, (NTM & 1) != 0>(a, p, s, chi, lane); break;
                default: break;
            }
        }
        return;
    }
    double nrm[1] = {0.0};
    cplx<T> acc[12];
    if (w == 0 && active) {
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {0, 0};
        add_staged<0, P, DAG>(chi, lane, acc);
        add_staged<1, P, DAG>(chi, lane, acc);
        add_staged<2, P, DAG>(chi, lane, acc);
        add_staged<3, P, DAG>(chi, lane, acc);
        add_staged<4, P, DAG>(chi, lane, acc);
        add_staged<5, P, DAG>(chi, lane, acc);
        add_staged<6, P, DAG>(chi, lane, acc);
        add_staged<7, P, DAG>(chi, lane, acc);
        if (!early) load_y<P, HASY, CG == CG_DIR_Y>(a, p, s, y);
        if constexpr (std::is_void<CT>::value)
            nrm[0] = hop_epilogue<P, HASY, NORM, (NTM & 1) != 0>(a, p, s, y, acc, NORM == 2 ? alpha : 0.0);
    }
    if constexpr (!std::is_void<CT>::value) {
        static_assert(canon_stage_bytes<spinor_granules<CT>()>() <= sizeof(chi), "the tile fits the staging");
        hop_canon<CT, P, HASY, 512>(a, p, s, w == 0 && active, y, acc, reinterpret_cast<v4u *>(chi));
    }
    if constexpr (NORM) {
        // wave 0 holds every site of the tile: a wave reduction suffices and
        // the other waves leave after the staging barrier
        if (w == 0) {
            const double t = wave_sum(nrm[0]);
            if (lane == 0 && blk < a.g.ntiles) a.partial[blk] = t;
        }
    }
}

constexpr int hop_shape(int prec) {
    return prec == LQCD_F64 ? LQCD_HOP_SHAPE_F64 : prec == LQCD_F32 ? LQCD_HOP_SHAPE_F32
                                                                     : LQCD_HOP_SHAPE_F16;
}

// Instances exist for the launches that the rules of hop_launch make.  Links of
// lattices below 2^17 sites per parity never exceed the Infinity Cache, so the
// row-parallel and the solver's small-lattice instances have no streamed-link
// form (NTM bit 1), nor have small ones with a norm (t-region launches, which
// are small at any size, have none); a build that forces the hints takes the
// general instance there.
template <int P, int LK, bool DAG, bool HASY, int NORM, int NTM, bool HALO>
static void launch_halo(const HopArgs &a, dim3 grid, hipStream_t st) {
    constexpr bool streamed = (NTM & 2) != 0;
    if constexpr (DAG && NORM == 1) {
        // (no other adjoint hop leaves a norm)
        if constexpr (P == LQCD_F64 && HASY && !HALO) {
#define LQCD_RESID(PI)                                                                             \
    if (a.cg == CG_RESID + PI) {                                                                   \
        if (!streamed && a.small) hop4_kernel<P, LK, DAG, HASY, NORM, NTM, HALO, void, CG_RESID + PI, streamed><<<grid, 256, a.lds_extra, st>>>(a); \
        else hop4_kernel<P, LK, DAG, HASY, NORM, NTM, HALO, void, CG_RESID + PI, true><<<grid, 256, a.lds_extra, st>>>(a); \
        return;                                                                                    \
    }
            LQCD_RESID(LQCD_F64)
            LQCD_RESID(LQCD_F32)
            LQCD_RESID(LQCD_F16)
#undef LQCD_RESID
        }
        return;
    } else {
        if constexpr (P != LQCD_F16 && !DAG && !HALO && (!streamed || LQCD_HOP_STREAM >= 0) && (HASY ? NORM == 1 : NORM == 0)) {
            constexpr int role = HASY ? CG_DIR_Y : CG_DIR_IN;
            if (a.cg == role) {
                if constexpr (hop_shape(P) == 8) hop8_kernel<P, LK, DAG, HASY, NORM, NTM, !HASY && P == LQCD_F32, HALO, void, role, false><<<grid, 512, 0, st>>>(a);
                else hop4_kernel<P, LK, DAG, HASY, NORM, NTM, HALO, void, role, false><<<grid, 256, 0, st>>>(a);
                return;
            }
        }
        if constexpr (DAG && !HASY && !NORM && !HALO) {
            if (a.cg == CG_PRE) {
                if constexpr (hop_shape(P) == 8) {
                    if constexpr (!streamed) {
                        if (a.rows) {
                            hop8_kernel<P, LK, DAG, HASY, NORM, NTM, true, HALO, void, CG_PRE, false><<<grid, 512, 0, st>>>(a);
                            return;
                        }
                    }
                    hop8_kernel<P, LK, DAG, HASY, NORM, NTM, false, HALO, void, CG_PRE><<<grid, 512, 0, st>>>(a);
                } else {
                    hop4_kernel<P, LK, DAG, HASY, NORM, NTM, HALO, void, CG_PRE><<<grid, 256, a.lds_extra, st>>>(a);
                }
                return;
            }
        }
        constexpr bool small = HALO || !(streamed && NORM);
        if constexpr (hop_shape(P) == 1) {
            hop1_kernel<P, LK, DAG, HASY, NORM, NTM, HALO><<<grid, 64, 0, st>>>(a);
        } else if constexpr (hop_shape(P) == 8) {
            if constexpr (P == LQCD_F32 && !HASY && !NORM && !streamed) {
                if (a.rows) {
                    hop8_kernel<P, LK, DAG, HASY, NORM, NTM, true, HALO, void, CG_NONE, false><<<grid, 512, 0, st>>>(a);
                    return;
                }
            }
            if (small && a.small) hop8_kernel<P, LK, DAG, HASY, NORM, NTM, false, HALO, void, CG_NONE, !small><<<grid, 512, 0, st>>>(a);
            else hop8_kernel<P, LK, DAG, HASY, NORM, NTM, false, HALO, void, CG_NONE, !HALO><<<grid, 512, 0, st>>>(a);
        } else {
            if constexpr (!HALO && LQCD_HOP_TMARCH > 0) {
                if (a.tseg > 0) {
                    hop4t_kernel<P, LK, DAG, HASY, NORM, NTM><<<grid, 256, a.lds_extra, st>>>(a);
                    return;
                }
            }
            if (small && a.small) hop4_kernel<P, LK, DAG, HASY, NORM, NTM, HALO, void, CG_NONE, !small><<<grid, 256, a.lds_extra, st>>>(a);
            else hop4_kernel<P, LK, DAG, HASY, NORM, NTM, HALO, void, CG_NONE, !HALO><<<grid, 256, a.lds_extra, st>>>(a);
        }
    }
}

// Boundary-slice launches (faces given) have no norm partial; the face
// variants exist only for the other combinations.
template <int P, int LK, bool DAG, bool HASY, int NORM, int NTM>
static void launch_nt(const HopArgs &a, dim3 grid, hipStream_t st) {
    if constexpr (!NORM) {
        if (a.face[0] != nullptr) {
            launch_halo<P, LK, DAG, HASY, NORM, NTM, true>(a, grid, st);
            return;
        }
    }
    launch_halo<P, LK, DAG, HASY, NORM, NTM, false>(a, grid, st);
}

// The cache hints are template arguments: a run-time choice between two
// otherwise identical load or store sequences gets merged by the compiler,
// which then drops the hint.  The stores' is the build's, the links' the
// launch's (LQCD_HOP_STREAM: both the build's).
template <int P, int LK, bool DAG, bool HASY, int NORM>
static void launch_shape(const HopArgs &a, dim3 grid, hipStream_t st) {
    constexpr int hint = LQCD_HOP_STREAM >= 0 ? LQCD_HOP_STREAM & 3 : OUT_NT ? 1 : 0;
    if constexpr (LQCD_HOP_STREAM < 0 && LQCD_LINK_NT) {
        if (a.stream & 2) {
            launch_nt<P, LK, DAG, HASY, NORM, hint | 2>(a, grid, st);
            return;
        }
    }
    launch_nt<P, LK, DAG, HASY, NORM, hint>(a, grid, st);
}

// norm: 0 none, 1 |out|^2 block partials (with a y term), 2 CG update (needs
// the y term; the solver applies it on the adjoint hop only)
template <int P, int LK, bool DAG>
static void launch_p(const HopArgs &a, bool hasy, int norm, dim3 grid, hipStream_t st) {
    if (hasy) {
        if (norm == 1) launch_shape<P, LK, DAG, true, 1>(a, grid, st);
        else if constexpr (DAG) {
            if (norm == 2) launch_shape<P, LK, DAG, true, 2>(a, grid, st);
            else launch_shape<P, LK, DAG, true, 0>(a, grid, st);
        } else {
            launch_shape<P, LK, DAG, true, 0>(a, grid, st);
        }
    } else {
        launch_shape<P, LK, DAG, false, 0>(a, grid, st);
    }
}

// Canonical output (FP64 and FP32 storage, both parities): links and stores
// without hints, as a both-parity launch wants them.
template <int P, int LK, bool DAG, bool HASY, typename CT>
static void launch_canon_ct(const HopArgs &a, dim3 grid, hipStream_t st) {
    if constexpr (hop_shape(P) == 8) hop8_kernel<P, LK, DAG, HASY, 0, 0, false, false, CT><<<grid, 512, 0, st>>>(a);
    else hop4_kernel<P, LK, DAG, HASY, 0, 0, false, CT><<<grid, 256, a.lds_extra, st>>>(a);
}

template <int P, int LK, bool DAG>
static void launch_canon(const HopArgs &a, bool hasy, dim3 grid, hipStream_t st) {
    if (a.canon == 8) {
        if (hasy) launch_canon_ct<P, LK, DAG, true, double>(a, grid, st);
        else launch_canon_ct<P, LK, DAG, false, double>(a, grid, st);
    } else {
        if (hasy) launch_canon_ct<P, LK, DAG, true, float>(a, grid, st);
        else launch_canon_ct<P, LK, DAG, false, float>(a, grid, st);
    }
}

template <int P, int LK>
static void launch_l(const HopArgs &a, bool dag, bool hasy, int norm, dim3 grid, hipStream_t st) {
    if constexpr (P != LQCD_F16) {
        if (a.canon != 0) {
            if (dag) launch_canon<P, LK, true>(a, hasy, grid, st);
            else launch_canon<P, LK, false>(a, hasy, grid, st);
            return;
        }
    }
    if (dag) launch_p<P, LK, true>(a, hasy, norm, grid, st);
    else launch_p<P, LK, false>(a, hasy, norm, grid, st);
}

int hop_launch(const HopArgs &a0, int prec, int link, bool dag, int nparity, hipStream_t st,
               int region) {
    if (prec == LQCD_F16 && a0.g.ntiles > F16_MAX_TILES) return LQCD_EINVAL;
    HopArgs a = a0;
    if (region < 0) {
        a.brick = launch_brick(a.g, prec, nparity == 2 && LQCD_HOP_PAIRED ? 2
                                          : nparity == 1 && LQCD_BRICK_BAND_EO ? 1 : 0,
                               nparity == 2);
        a.bpp = brick_blocks(a.g, a.brick);
        a.face[0] = a.face[1] = nullptr;
    } else {
        // interior slices 1 .. Lt-2, or boundary slices 0 and Lt-1
        const int lt = a.g.L[3];
        const int nt = region == 0 ? lt - 2 : 2;
        if (nt <= 0) return LQCD_OK;
        a.bpp = (int64_t)nt * (a.g.st / TILE);
        a.brick = make_region_brick(a.g, brick_plan(a.g, prec), region == 0 ? 1 : 0,
                                    region == 0 ? 1 : lt - 1, nt);
        if (region == 0) a.face[0] = a.face[1] = nullptr;
        nparity = 1;
    }
    a.paired = nparity == 2 && LQCD_HOP_PAIRED;
    // row-parallel rebuild only where a launch is latency-bound (V/2 < 2^17:
    // 16^4 and smaller); from 24^4 up the single-wave rebuild is 0.5-2.5
    // points faster
    a.rows = LQCD_HOP_ROWS && a.g.vh < ((int64_t)1 << 17) && a.y[0] == nullptr &&
             a.y[1] == nullptr && a.partial == nullptr && a.cg != CG_UPDATE;
    const int64_t spinors = (int64_t)(nparity * half_spinor_bytes(a.g, prec));
    const int64_t links = (int64_t)gauge_bytes(a.g, prec, link);
    const bool out_nt = OUT_NT;
    // a both-parity launch reads every link twice (forward from its own site,
    // backward from the paired tile), so it keeps them cached
    const bool link_nt = LQCD_LINK_NT && !a.paired && spinors + links > INFINITY_CACHE_BYTES;
    a.stream = LQCD_HOP_STREAM >= 0 ? LQCD_HOP_STREAM : (out_nt ? 1 : 0) | (link_nt ? 2 : 0);
    a.lds_extra = LQCD_HOP_EXTRA_LDS >= 0 ? (uint32_t)LQCD_HOP_EXTRA_LDS : 0u;
    if (LQCD_HOP_EXTRA_LDS < 0 && prec == LQCD_F64 &&
        a.g.vh >= ((int64_t)1 << (a.paired      ? LQCD_HOP_F64_PAIRED_LDS_MIN_LOG2
                                  : region < 0 ? LQCD_HOP_F64_LDS_MIN_LOG2
                                               : LQCD_HOP_F64_REGION_LDS_MIN_LOG2))) {
        const bool plain = a.brick.lz == 1 && a.g.vh >= ((int64_t)1 << LQCD_BRICK_MIN_LOG2);
        const bool wide = a.brick.lz == 0 && a.g.st * (2 * 3 * 192 / 8) > F64_SLAB_TWO_BYTES;
        const bool two = a.paired && link == 18 && (plain || wide);
        a.lds_extra = two ? F64_LDS_TWO : F64_LDS_THREE;
    }
    const bool short_launch = a.g.vh < ((int64_t)1 << BIG_MIN_LOG2) || region >= 0;
    a.rev = LQCD_HOP_ZIGZAG && nparity == 1 && !short_launch && a.par0 == LQCD_ODD;
    // binary16 hops, bound by their instructions, take the instances without
    // the other orders wherever they use none of them (us, with the orders ->
    // without: M 32^4 56.6 -> 56.3, 24^4 17.4 -> 17.3, Mhat 32^4 61.1 -> 60.8)
    a.small = short_launch || (prec == LQCD_F16 && !a.rev && a.brick.lz != 0);
    dim3 grid((unsigned)(a.bpp * nparity));
    // t-march launches (4-way shape, one parity, whole lattice, whole tiles
    // per t-slice in a multiple of 8 columns; the solver's other roles are
    // those of the 4-way form): one block per column and segment of tseg slices
    a.tseg = 0;
    if (LQCD_HOP_TMARCH > 0 && hop_shape(prec) == 4 && nparity == 1 && region < 0 &&
        (a.cg == CG_NONE || a.cg == CG_UPDATE) &&
        a.g.vh >= ((int64_t)1 << LQCD_HOP_TMARCH_MIN_LOG2) && a.g.st % TILE == 0 &&
        (a.g.st / TILE) % 8 == 0) {
        a.tseg = LQCD_HOP_TMARCH;
        const int64_t nseg = (a.g.L[3] + a.tseg - 1) / a.tseg;
        grid = dim3((unsigned)((a.g.st / TILE) * nseg));
        a.lds_extra = LQCD_HOP_EXTRA_LDS >= 0 ? (uint32_t)LQCD_HOP_EXTRA_LDS : 0u;
    }
    // a launch counts its work items in 32 bits and drops what is beyond
    if ((int64_t)grid.x * (hop_shape(prec) == 8 ? 512 : 256) > UINT32_MAX) return LQCD_EINVAL;
    a.nblk = grid.x;
    const bool hasy = a.y[0] != nullptr || a.y[1] != nullptr;
    const int norm = a.cg == CG_UPDATE ? 2 : a.partial != nullptr ? 1 : 0;
    const bool dir = a.cg == CG_DIR_IN || a.cg == CG_DIR_Y;
    // (of the hops that leave a norm, the adjoint ones are those of CG_RESID)
    if (norm == 1 && (!hasy || (dag && a.cg < CG_RESID))) return LQCD_EINVAL;
    if (dir && (prec == LQCD_F16 || dag || !a.sums || !a.sc || !a.p_old ||
                ((a.stream & 2) && LQCD_HOP_STREAM < 0)))
        return LQCD_EINVAL;
    if (a.cg == CG_DIR_IN && (hasy || norm)) return LQCD_EINVAL;
    if (a.cg == CG_DIR_Y && (!hasy || norm != 1 || !a.p_new || !a.x || a.p_new == a.p_old)) return LQCD_EINVAL;
    if ((a.cg == CG_PRE || a.cg == CG_UPDATE) && (!dag || !a.sums || !a.sc)) return LQCD_EINVAL;
    if (a.cg >= CG_RESID && (prec != LQCD_F64 || !dag || !hasy || norm != 1 || !a.rhs || !a.stored))
        return LQCD_EINVAL;
    if (a.cg == CG_UPDATE && (!hasy || !a.partial)) return LQCD_EINVAL;
    // a pre-summing launch has a block for every group
    if (a.cg == CG_PRE && (hasy || norm || !a.groups || (int64_t)a.n_groups > a.bpp)) return LQCD_EINVAL;
    if (prec == LQCD_F64) {
        if (link == 18) launch_l<LQCD_F64, 18>(a, dag, hasy, norm, grid, st);
        else launch_l<LQCD_F64, 12>(a, dag, hasy, norm, grid, st);
    } else if (prec == LQCD_F32) {
        if (link == 18) launch_l<LQCD_F32, 18>(a, dag, hasy, norm, grid, st);
        else launch_l<LQCD_F32, 12>(a, dag, hasy, norm, grid, st);
    } else {
        launch_l<LQCD_F16, 12>(a, dag, hasy, norm, grid, st);
    }
    return check_launch();
}

int64_t hop_partials(const Geom &g, int nparity) {
    return ((g.vh + HOP_SITES - 1) / HOP_SITES) * nparity;
}

}  // namespace lqcd

using namespace lqcd;

static int validate_hop(const lqcd_geom_t *gg, Geom *g, const void *out, const void *in,
                        const void *U, int prec, int link) {
    if (!make_geom(gg, g)) return LQCD_EINVAL;
    if (!valid_link(prec, link)) return LQCD_EINVAL;
    if (!out || !in || !U) return LQCD_EINVAL;
    if (((uintptr_t)out | (uintptr_t)in | (uintptr_t)U) & 15) return LQCD_EINVAL;
    if (out == in) return LQCD_EINVAL;
    return LQCD_OK;
}

static int full_hop(const lqcd_geom_t *gg, void *out, const void *in, const void *y, const void *U,
                    double alpha, double beta, int prec, int link, bool dag, void *stream,
                    int canon_real = 0) {
    Geom g;
    int rc = validate_hop(gg, &g, out, in, U, prec, link);
    if (rc) return rc;
    if (y && ((uintptr_t)y & 15)) return LQCD_EINVAL;
    const size_t hb = half_spinor_bytes(g, prec);
    HopArgs a{};
    a.g = g;
    a.U = (const char *)U;
    a.alpha = alpha;
    a.beta = beta;
    a.par0 = 0;
    a.canon = canon_real;
    // output parity p reads the other parity's half of the input
    a.out[0] = (char *)out;
    a.out[1] = (char *)out + hb;
    a.in[0] = (const char *)in + hb;
    a.in[1] = (const char *)in;
    a.y[0] = y ? (const char *)y : nullptr;
    a.y[1] = y ? (const char *)y + hb : nullptr;
    a.partial = nullptr;
    return hop_launch(a, prec, link, dag, 2, (hipStream_t)stream);
}

extern "C" int lqcd_dslash(const lqcd_geom_t *g, void *out, const void *in, const void *y,
                           const void *U, double alpha, double beta, int prec, int link,
                           void *stream) {
    return full_hop(g, out, in, y, U, alpha, beta, prec, link, false, stream);
}

extern "C" int lqcd_dslash_dagger(const lqcd_geom_t *g, void *out, const void *in,
                                  const void *y, const void *U, double alpha, double beta,
                                  int prec, int link, void *stream) {
    return full_hop(g, out, in, y, U, alpha, beta, prec, link, true, stream);
}

extern "C" int lqcd_dslash_canonical(const lqcd_geom_t *g, void *out_canon, int canon_prec,
                                     const void *in, const void *y, const void *U, double alpha,
                                     double beta, int dagger, int prec, int link, void *stream) {
    if (canon_prec != LQCD_F64 && canon_prec != LQCD_F32) return LQCD_EINVAL;
    if (prec != LQCD_F64 && prec != LQCD_F32) return LQCD_EINVAL;
    if (out_canon == y) return LQCD_EINVAL;  // (out_canon == NULL is refused either way)
    return full_hop(g, out_canon, in, y, U, alpha, beta, prec, link, dagger != 0, stream,
                    canon_prec == LQCD_F64 ? 8 : 4);
}

static int eo_hop(const lqcd_geom_t *gg, int out_par, void *out, const void *in, const void *y,
                  const void *U, double alpha, double beta, int dagger, int prec, int link,
                  void *stream) {
    Geom g;
    int rc = validate_hop(gg, &g, out, in, U, prec, link);
    if (rc) return rc;
    if (y && ((uintptr_t)y & 15)) return LQCD_EINVAL;
    HopArgs a{};
    a.g = g;
    a.U = (const char *)U;
    a.alpha = alpha;
    a.beta = beta;
    a.par0 = out_par;
    a.out[out_par] = (char *)out;
    a.in[out_par] = (const char *)in;
    a.y[out_par] = (const char *)y;
    a.partial = nullptr;
    return hop_launch(a, prec, link, dagger != 0, 1, (hipStream_t)stream);
}

extern "C" int lqcd_meo(const lqcd_geom_t *g, void *out_e, const void *in_o, const void *y_e,
                        const void *U, double alpha, double beta, int dagger, int prec, int link,
                        void *stream) {
    return eo_hop(g, LQCD_EVEN, out_e, in_o, y_e, U, alpha, beta, dagger, prec, link, stream);
}

extern "C" int lqcd_moe(const lqcd_geom_t *g, void *out_o, const void *in_e, const void *y_o,
                        const void *U, double alpha, double beta, int dagger, int prec, int link,
                        void *stream) {
    return eo_hop(g, LQCD_ODD, out_o, in_e, y_o, U, alpha, beta, dagger, prec, link, stream);
}

extern "C" int lqcd_hop_region(const lqcd_geom_t *gg, int out_par, int region, void *out,
                               const void *in, const void *y, const void *U,
                               const void *face_fwd, const void *face_bwd, double alpha,
                               double beta, int dagger, int prec, int link, void *stream) {
    Geom g;
    int rc = validate_hop(gg, &g, out, in, U, prec, link);
    if (rc) return rc;
    if (out_par != LQCD_EVEN && out_par != LQCD_ODD) return LQCD_EINVAL;
    if (region != 0 && region != 1) return LQCD_EINVAL;
    if (g.st % TILE != 0) return LQCD_EINVAL;  // t-slices must be whole tiles
    if (y && ((uintptr_t)y & 15)) return LQCD_EINVAL;
    if (region == 1 && (!face_fwd || !face_bwd || (((uintptr_t)face_fwd | (uintptr_t)face_bwd) & 15)))
        return LQCD_EINVAL;
    HopArgs a{};
    a.g = g;
    a.U = (const char *)U;
    a.alpha = alpha;
    a.beta = beta;
    a.par0 = out_par;
    a.out[out_par] = (char *)out;
    a.in[out_par] = (const char *)in;
    a.y[out_par] = (const char *)y;
    a.partial = nullptr;
    a.face[0] = (const char *)face_fwd;
    a.face[1] = (const char *)face_bwd;
    return hop_launch(a, prec, link, dagger != 0, 1, (hipStream_t)stream, region);
}

extern "C" int lqcd_mhat(const lqcd_geom_t *g, void *out_e, const void *in_e, void *tmp_o,
                         const void *U, double kappa, int dagger, int prec, int link,
                         void *stream) {
    if (!tmp_o || tmp_o == in_e || tmp_o == out_e) return LQCD_EINVAL;
    // Mhat      = 1 - k^2 D_eo D_oe:              tmp = D_oe in,        out = in - k^2 D_eo tmp
    // Mhat^dag  = 1 - k^2 (D_oe)^dag (D_eo)^dag:  tmp = (D_eo)^dag in,  out = in - k^2 (D_oe)^dag tmp
    int rc = lqcd_moe(g, tmp_o, in_e, nullptr, U, 1.0, 0.0, dagger, prec, link, stream);
    if (rc) return rc;
    return lqcd_meo(g, out_e, tmp_o, in_e, U, -kappa * kappa, 1.0, dagger, prec, link, stream);
}
