// Library information, geometry validation, size queries and the conversions
// between the canonical lexicographic arrays and the tiled internal layout.

#include <string.h>

#include "lqcd_internal.h"

namespace lqcd {

static thread_local char g_hip_error[256] = "";

void set_hip_error(hipError_t e) {
    const char *s = hipGetErrorString(e);
    strncpy(g_hip_error, s ? s : "unknown HIP error", sizeof(g_hip_error) - 1);
    g_hip_error[sizeof(g_hip_error) - 1] = 0;
}

int check_launch() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_hip_error(e);
        return LQCD_EHIP;
    }
    return LQCD_OK;
}

bool make_geom(const lqcd_geom_t *g, Geom *out) {
    if (!g || !out) return false;
    int64_t v = 1;
    for (int mu = 0; mu < 4; ++mu) {
        const int L = g->dims[mu];
        if (L < 2 || (L & 1) || L > (1 << 16)) return false;
        if (g->bc[mu] != 1 && g->bc[mu] != -1) return false;
        out->L[mu] = L;
        out->bc[mu] = g->bc[mu];
        v *= L;
    }
    if (v > ((int64_t)1 << 31)) return false;  // grid of one thread per site fits 32 bits
    out->lxh = g->dims[0] / 2;
    out->vh = v / 2;
    out->ntiles = (out->vh + TILE - 1) / TILE;
    out->sy = out->lxh;
    out->sz = out->sy * g->dims[1];
    out->st = out->sz * g->dims[2];
    out->dx = make_fastdiv((uint32_t)out->lxh);
    out->dy = make_fastdiv((uint32_t)g->dims[1]);
    out->dz = make_fastdiv((uint32_t)g->dims[2]);
    return true;
}

// ---------------------------------------------------------------------------
// pack / unpack kernels
// ---------------------------------------------------------------------------

// Both layouts are streamed at full width and the transposition between them
// happens in LDS: the canonical array is read (or written) as consecutive
// 16-byte granules by consecutive lanes, the tiles as 64-lane words.
// Checkerboard sites s of the two parities are the canonical pair 2s, 2s + 1,
// so the tile s/64 of both parities is one contiguous canonical run.  A pair
// (or, for a half field, a site) takes an odd number of granules in LDS, so
// lanes reading one granule each of consecutive pairs hit different banks.
// Pure streaming, bound by the memory system; a thread per site reading its
// own 192 (spinor) or 576 (links) bytes, as these kernels did before, touched
// 64 lines per load instruction.  Kernel times at 24^4, FP64 (us, before ->
// now): links in (18 reals) 91 -> 68, out 120 -> 56 (6.8 TB/s), spinor in
// 28 -> 26, out 34 -> 24 (5.4 TB/s); FP32 at 16^4: 8.2 -> 7.8, 15.7 -> 9.1,
// 4.7 -> 4.4, 5.9 -> 4.4.

constexpr int SPINOR_BLOCK = 128;  // sites per block: 64 pairs, or 128 sites of one parity
constexpr int GAUGE_PAIRS = 32;    // pairs per block, one thread per link

// One block of a spinor conversion: the pairs (HALF: the sites of parity
// `par`) s0, s0 + 1, ... as LDS slots, and this thread's own site.
template <typename CT, bool HALF>
struct SpinorBlock {
    static constexpr int GS = spinor_granules<CT>();
    static constexpr int SLOTS = HALF ? SPINOR_BLOCK : SPINOR_BLOCK / 2;
    static constexpr int PER = HALF ? GS : 2 * GS;  // granules of a slot
    static constexpr int STRIDE = PER + 1;          // odd, in LDS
    static_assert(STRIDE & 1, "slots an odd number of granules apart");

    int64_t s0;
    int count;  // slots in use
    int par;    // this thread's site: parity, slot and its granule in LDS
    int slot;
    int own;

    __device__ __forceinline__ SpinorBlock(const Geom &g, int subset) {
        const int tid = threadIdx.x;
        s0 = (int64_t)blockIdx.x * SLOTS;
        count = (int)(g.vh - s0 < SLOTS ? g.vh - s0 : SLOTS);
        slot = HALF ? tid : tid & (SLOTS - 1);
        par = HALF ? subset : tid / SLOTS;
        // the site of parity p in its pair is the one with x parity p ^ row
        own = slot * STRIDE + (HALF ? 0 : GS * (par ^ row_parity(g, (uint32_t)(s0 + slot))));
    }
    __device__ __forceinline__ int granules() const { return count * PER; }
    // canonical granule of the block's granule i
    __device__ __forceinline__ int64_t canon(const Geom &g, int i) const {
        if constexpr (!HALF) return s0 * PER + i;
        const int64_t s = s0 + i / GS;
        return (2 * s + (par ^ row_parity(g, (uint32_t)s))) * GS + i % GS;
    }
    __device__ __forceinline__ static int lds(int i) { return i / PER * STRIDE + i % PER; }
};

template <typename CT, int P, bool HALF>
__global__ __launch_bounds__(SPINOR_BLOCK) void pack_spinor_k(Geom g, char *dst, const v4u *src,
                                                              int subset, int64_t hb) {
    using T = typename real_of<P>::type;
    using B = SpinorBlock<CT, HALF>;
    __shared__ v4u stage[B::SLOTS * B::STRIDE];
    const B b(g, subset);
    const int n = b.granules();
    v4u q[B::GS];
#pragma unroll
    for (int j = 0; j < B::GS; ++j) {
        // the last block's surplus threads read its last granule again
        const int i = j * SPINOR_BLOCK + (int)threadIdx.x;
        q[j] = src[b.canon(g, i < n ? i : n - 1)];
    }
#pragma unroll
    for (int j = 0; j < B::GS; ++j) stage[B::lds(j * SPINOR_BLOCK + (int)threadIdx.x)] = q[j];
    __syncthreads();
    if (b.slot >= b.count) return;
    cplx<T> v[12];
    const CT *s = reinterpret_cast<const CT *>(stage + b.own);
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = {(T)s[2 * k], (T)s[2 * k + 1]};
    store_spinor<P>(dst + (HALF ? 0 : b.par * hb), b.s0 + b.slot, v);
}

template <typename CT, int P, bool HALF>
__global__ __launch_bounds__(SPINOR_BLOCK) void unpack_spinor_k(Geom g, v4u *dst, const char *src,
                                                                int subset, int64_t hb) {
    using T = typename real_of<P>::type;
    using B = SpinorBlock<CT, HALF>;
    __shared__ v4u stage[B::SLOTS * B::STRIDE];
    const B b(g, subset);
    if (b.slot < b.count) {
        cplx<T> v[12];
        load_spinor<P>(src + (HALF ? 0 : b.par * hb), b.s0 + b.slot, v);
        CT *d = reinterpret_cast<CT *>(stage + b.own);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            d[2 * k] = (CT)v[k].re;
            d[2 * k + 1] = (CT)v[k].im;
        }
    }
    __syncthreads();
    const int n = b.granules();
#pragma unroll
    for (int j = 0; j < B::GS; ++j) {
        const int i = j * SPINOR_BLOCK + (int)threadIdx.x;
        if (i < n) dst[b.canon(g, i)] = stage[B::lds(i)];
    }
}

// One block of a link conversion: GAUGE_PAIRS pairs, thread = (direction,
// parity, pair), so a wave holds one direction of both parities' sites.
template <typename CT>
struct GaugeBlock {
    static constexpr int THREADS = GAUGE_PAIRS * 8;
    static constexpr int GS = gauge_granules<CT>();
    static constexpr int STRIDE = 2 * GS + 1;
    static constexpr int STEPS = (GAUGE_PAIRS * 2 * GS + THREADS - 1) / THREADS;

    int64_t s0;
    int count, pair, par, mu;
    int own;  // this thread's link in LDS, in reals of CT

    __device__ __forceinline__ explicit GaugeBlock(const Geom &g) {
        const int tid = threadIdx.x;
        s0 = (int64_t)blockIdx.x * GAUGE_PAIRS;
        count = (int)(g.vh - s0 < GAUGE_PAIRS ? g.vh - s0 : GAUGE_PAIRS);
        pair = tid % GAUGE_PAIRS;
        par = tid / GAUGE_PAIRS & 1;
        mu = tid / (2 * GAUGE_PAIRS);
        own = (pair * STRIDE + GS * (par ^ row_parity(g, (uint32_t)(s0 + pair)))) * (WORD / (int)sizeof(CT)) + mu * 18;
    }
    __device__ __forceinline__ int granules() const { return count * 2 * GS; }
    __device__ __forceinline__ static int lds(int i) { return i / (2 * GS) * STRIDE + i % (2 * GS); }
};

template <typename CT, int P, int LK>
__global__ __launch_bounds__(GaugeBlock<CT>::THREADS) void pack_gauge_k(Geom g, char *dst,
                                                                        const v4u *src) {
    using T = typename real_of<P>::type;
    using B = GaugeBlock<CT>;
    __shared__ v4u stage[GAUGE_PAIRS * B::STRIDE];
    const B b(g);
    const int n = b.granules();
    src += b.s0 * 2 * B::GS;
    v4u q[B::STEPS];
#pragma unroll
    for (int j = 0; j < B::STEPS; ++j) {
        const int i = j * B::THREADS + (int)threadIdx.x;
        q[j] = src[i < n ? i : n - 1];
    }
#pragma unroll
    for (int j = 0; j < B::STEPS; ++j) {
        const int i = j * B::THREADS + (int)threadIdx.x;
        if (i < n) stage[B::lds(i)] = q[j];
    }
    __syncthreads();
    if (b.pair >= b.count) return;
    cplx<T> u[9];
    const CT *s = reinterpret_cast<const CT *>(stage) + b.own;
#pragma unroll
    for (int k = 0; k < 9; ++k) u[k] = {(T)s[2 * k], (T)s[2 * k + 1]};
    store_link<P, LK>(dst, g.ntiles, b.par, b.s0 + b.pair, b.mu, u);
}

template <typename CT, int P, int LK>
__global__ __launch_bounds__(GaugeBlock<CT>::THREADS) void unpack_gauge_k(Geom g, v4u *dst,
                                                                          const char *src) {
    using T = typename real_of<P>::type;
    using B = GaugeBlock<CT>;
    __shared__ v4u stage[GAUGE_PAIRS * B::STRIDE];
    const B b(g);
    if (b.pair < b.count) {
        cplx<T> u[9];
        load_link<P, LK>(src, g.ntiles, b.par, b.s0 + b.pair, b.mu, u);
        CT *d = reinterpret_cast<CT *>(stage) + b.own;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            d[2 * k] = (CT)u[k].re;
            d[2 * k + 1] = (CT)u[k].im;
        }
    }
    __syncthreads();
    const int n = b.granules();
    dst += b.s0 * 2 * B::GS;
#pragma unroll
    for (int j = 0; j < B::STEPS; ++j) {
        const int i = j * B::THREADS + (int)threadIdx.x;
        if (i < n) dst[i] = stage[B::lds(i)];
    }
}

}  // namespace lqcd

using namespace lqcd;

// ---------------------------------------------------------------------------
// library information and sizes
// ---------------------------------------------------------------------------

extern "C" int lqcd_version(void) { return 10000; }

extern "C" const char *lqcd_strerror(int status) {
    switch (status) {
        case LQCD_OK: return "ok";
        case LQCD_EINVAL: return "invalid argument (geometry, pointer, alignment or precision/link combination)";
        case LQCD_EHIP: return "HIP runtime or launch error";
        case LQCD_ENOCONV: return "solver did not converge within maxiter";
        case LQCD_ENAN: return "non-finite residual";
        case LQCD_ESMALL: return "workspace (or static scratch) too small";
        default: return "unknown status";
    }
}

extern "C" const char *lqcd_last_hip_error(void) { return g_hip_error; }

extern "C" size_t lqcd_spinor_bytes(const lqcd_geom_t *gg, int prec, int subset) {
    Geom g;
    if (!make_geom(gg, &g) || !valid_prec(prec)) return 0;
    if (subset != LQCD_EVEN && subset != LQCD_ODD && subset != LQCD_FULL) return 0;
    return half_spinor_bytes(g, prec) * (subset == LQCD_FULL ? 2 : 1);
}

extern "C" size_t lqcd_gauge_bytes(const lqcd_geom_t *gg, int prec, int link) {
    Geom g;
    if (!make_geom(gg, &g) || !valid_link(prec, link)) return 0;
    return gauge_bytes(g, prec, link);
}

// ---------------------------------------------------------------------------
// pack / unpack entry points
// ---------------------------------------------------------------------------

static bool aligned16(const void *p) { return p && (((uintptr_t)p) & 15) == 0; }

template <typename CT, bool PACK, bool HALF>
static void launch_spinor_p(const Geom &g, void *dst, const void *src, int prec, int subset,
                            hipStream_t st) {
    constexpr int slots = SpinorBlock<CT, HALF>::SLOTS;
    dim3 grid((unsigned)((g.vh + slots - 1) / slots)), block(SPINOR_BLOCK);
    const int64_t hb = (int64_t)half_spinor_bytes(g, prec);
#define LQCD_SPINOR_CASE(P)                                                                        \
    if (prec == P) {                                                                               \
        if (PACK) pack_spinor_k<CT, P, HALF><<<grid, block, 0, st>>>(g, (char *)dst, (const v4u *)src, subset, hb); \
        else unpack_spinor_k<CT, P, HALF><<<grid, block, 0, st>>>(g, (v4u *)dst, (const char *)src, subset, hb);    \
        return;                                                                                    \
    }
    LQCD_SPINOR_CASE(LQCD_F64)
    LQCD_SPINOR_CASE(LQCD_F32)
    LQCD_SPINOR_CASE(LQCD_F16)
#undef LQCD_SPINOR_CASE
}

template <typename CT, bool PACK>
static void launch_spinor(const Geom &g, void *dst, const void *src, int prec, int subset,
                          hipStream_t st) {
    if (subset == LQCD_FULL) launch_spinor_p<CT, PACK, false>(g, dst, src, prec, subset, st);
    else launch_spinor_p<CT, PACK, true>(g, dst, src, prec, subset, st);
}

static int spinor_args(const lqcd_geom_t *gg, Geom *g, const void *a, const void *b,
                       int canon_prec, int prec, int subset) {
    if (!make_geom(gg, g)) return LQCD_EINVAL;
    if (!valid_prec(prec)) return LQCD_EINVAL;
    if (canon_prec != LQCD_F64 && canon_prec != LQCD_F32) return LQCD_EINVAL;
    if (subset != LQCD_EVEN && subset != LQCD_ODD && subset != LQCD_FULL) return LQCD_EINVAL;
    if (!aligned16(a) || !aligned16(b)) return LQCD_EINVAL;
    return LQCD_OK;
}

extern "C" int lqcd_pack_spinor(const lqcd_geom_t *gg, void *dst, const void *src_canon,
                                int canon_prec, int prec, int subset, void *stream) {
    Geom g;
    int rc = spinor_args(gg, &g, dst, src_canon, canon_prec, prec, subset);
    if (rc) return rc;
    if (canon_prec == LQCD_F64) launch_spinor<double, true>(g, dst, src_canon, prec, subset, (hipStream_t)stream);
    else launch_spinor<float, true>(g, dst, src_canon, prec, subset, (hipStream_t)stream);
    return check_launch();
}

extern "C" int lqcd_unpack_spinor(const lqcd_geom_t *gg, void *dst_canon, const void *src,
                                  int canon_prec, int prec, int subset, void *stream) {
    Geom g;
    int rc = spinor_args(gg, &g, dst_canon, src, canon_prec, prec, subset);
    if (rc) return rc;
    if (canon_prec == LQCD_F64) launch_spinor<double, false>(g, dst_canon, src, prec, subset, (hipStream_t)stream);
    else launch_spinor<float, false>(g, dst_canon, src, prec, subset, (hipStream_t)stream);
    return check_launch();
}

template <typename CT, bool PACK>
static void launch_gauge(const Geom &g, void *dst, const void *src, int prec, int link,
                         hipStream_t st) {
    dim3 grid((unsigned)((g.vh + GAUGE_PAIRS - 1) / GAUGE_PAIRS)), block(GaugeBlock<CT>::THREADS);
#define LQCD_GAUGE_CASE(P, LK)                                                                   \
    if (prec == P && link == LK) {                                                              \
        if (PACK) pack_gauge_k<CT, P, LK><<<grid, block, 0, st>>>(g, (char *)dst, (const v4u *)src); \
        else unpack_gauge_k<CT, P, LK><<<grid, block, 0, st>>>(g, (v4u *)dst, (const char *)src);   \
        return;                                                                                 \
    }
    LQCD_GAUGE_CASE(LQCD_F64, 18)
    LQCD_GAUGE_CASE(LQCD_F64, 12)
    LQCD_GAUGE_CASE(LQCD_F32, 18)
    LQCD_GAUGE_CASE(LQCD_F32, 12)
    LQCD_GAUGE_CASE(LQCD_F16, 12)
#undef LQCD_GAUGE_CASE
}

extern "C" int lqcd_pack_gauge(const lqcd_geom_t *gg, void *dst, const void *src_canon,
                               int canon_prec, int prec, int link, void *stream) {
    Geom g;
    if (!make_geom(gg, &g) || !valid_link(prec, link)) return LQCD_EINVAL;
    if (canon_prec != LQCD_F64 && canon_prec != LQCD_F32) return LQCD_EINVAL;
    if (!aligned16(dst) || !aligned16(src_canon)) return LQCD_EINVAL;
    if (canon_prec == LQCD_F64) launch_gauge<double, true>(g, dst, src_canon, prec, link, (hipStream_t)stream);
    else launch_gauge<float, true>(g, dst, src_canon, prec, link, (hipStream_t)stream);
    return check_launch();
}

extern "C" int lqcd_unpack_gauge(const lqcd_geom_t *gg, void *dst_canon, const void *src,
                                 int canon_prec, int prec, int link, void *stream) {
    Geom g;
    if (!make_geom(gg, &g) || !valid_link(prec, link)) return LQCD_EINVAL;
    if (canon_prec != LQCD_F64 && canon_prec != LQCD_F32) return LQCD_EINVAL;
    if (!aligned16(dst_canon) || !aligned16(src)) return LQCD_EINVAL;
    if (canon_prec == LQCD_F64) launch_gauge<double, false>(g, dst_canon, src, prec, link, (hipStream_t)stream);
    else launch_gauge<float, false>(g, dst_canon, src, prec, link, (hipStream_t)stream);
    return check_launch();
}
