// BLAS-1 on internal spinor fields: inner products and norms with
// deterministic wave64 -> block -> grid reductions, y = a x + b y, and
// precision conversion.  FP64 and FP32 fields are reduced and updated as runs of
// 16-byte words (the sum of a word's products in the field's arithmetic, all
// above it in FP64), binary16 fields and conversions site by site; a FULL
// field is the even half followed by the odd half.

#include <mutex>

#include "lqcd_internal.h"
#include "reduce.h"
#include "blas.h"
#include "grid.h"
#include "mail.h"

namespace lqcd {

constexpr int RED_BLOCK = 256;

// Ablation switch: 1 replaces the wave64 -> block -> fixed-order grid
// reduction by one FP64 atomic add per thread into the result (which is then
// order-dependent, i.e. not reproducible bit for bit).
#ifndef LQCD_REDUCE_ATOMIC
#define LQCD_REDUCE_ATOMIC 0
#endif

int64_t reduce_blocks(const Geom &g, int nhalf) { return (g.vh * nhalf + RED_BLOCK - 1) / RED_BLOCK; }

// At most this many blocks walk a field, so a final sum is short and every
// block has work for a while.
constexpr int64_t RED_GRID = 2048;
int64_t reduce_grid(const Geom &g, int nhalf) {
    const int64_t n = reduce_blocks(g, nhalf);
    return n < RED_GRID ? n : RED_GRID;
}

// One 16-byte word of a FP64 (one complex) or FP32 field (two).
template <int P, bool DOT>
__device__ __forceinline__ void reduce_word(v4u wa, v4u wb, double acc[2]) {
    using T = typename real_of<P>::type;
    constexpr int n = P == LQCD_F64 ? 1 : 2;
    cplx<T> a[n], b[n];
    __builtin_memcpy(a, &wa, 16);
    __builtin_memcpy(b, &wb, 16);
    T re = 0, im = 0;
#pragma unroll
    for (int k = 0; k < n; ++k) {
        if constexpr (DOT) {
            const cplx<T> z = cmul_conj(a[k], b[k]);
            re += z.re;
            im += z.im;
        } else {
            re += norm2(a[k]);
        }
    }
    acc[0] += (double)re;
    acc[1] += (double)im;
}

// <a, b> or |a|^2 over `nhalf` half fields of ntiles tiles, vh sites each.
// FP64 and FP32 fields are read as one run of 16-byte words, one word per
// thread and load, two of each field in flight (site by site a wave took all
// the words of one tile); lanes past the last site of a half are left out.
// binary16 fields are read site by site, for the scale.  Whole call at 32^4,
// full field (us, before -> now, the posted result and the shorter final sum
// included): <a, b> FP64 98 -> 86, FP32 60.6 -> 49, |a|^2 FP64 61 -> 51, FP32 47
// -> 36; at 8^4 31.5 -> 21.  Four or eight words in flight, or 1024 or 4096
// blocks: 6-15 us more for the first.
template <int P, bool DOT, bool RAGGED>
__global__ __launch_bounds__(RED_BLOCK) void reduce_k(const char *a, const char *b, int64_t vh,
                                                      int64_t ntiles, int nhalf, int64_t hb, double *partial) {
    using T = typename real_of<P>::type;
    const int64_t step = (int64_t)gridDim.x * RED_BLOCK;
    int64_t i = (int64_t)blockIdx.x * RED_BLOCK + threadIdx.x;
    double acc[2] = {0.0, 0.0};
    if constexpr (P == LQCD_F16) {
        for (; i < vh * nhalf; i += step) {
            const int64_t off = i >= vh ? hb : 0, s = i >= vh ? i - vh : i;
            cplx<T> va[12], vb[12];
            load_spinor<P>(a + off, s, va);
            if constexpr (DOT) load_spinor<P>(b + off, s, vb);
            T re = 0, im = 0;
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                if constexpr (DOT) {
                    const cplx<T> z = cmul_conj(va[k], vb[k]);
                    re += z.re;
                    im += z.im;
                } else {
                    re += norm2(va[k]);
                }
            }
            acc[0] += (double)re;
            acc[1] += (double)im;
        }
    } else {
        constexpr int NW = spinor_tile_bytes(P) / WORD;  // words of a tile
        const int64_t n = nhalf * ntiles * NW;
        const v4u *wa = reinterpret_cast<const v4u *>(a), *wb = reinterpret_cast<const v4u *>(DOT ? b : a);
        // (blocks are whole waves, so the lane of word i is the thread's)
        auto mine = [&](int64_t j) {
            if constexpr (LQCD_LAYOUT_AOS && RAGGED) {
                const int64_t site = j * (WORD / (P == LQCD_F64 ? 192 : 96.0));
                return (site >= ntiles * TILE ? site - ntiles * TILE : site) < vh;
            }
            if constexpr (!RAGGED) return true;
            int64_t tile = j / NW;
            if (tile >= ntiles) tile -= ntiles;
            return tile * TILE + (j & (TILE - 1)) < vh;
        };
        constexpr int U = 2;
        for (; i + (U - 1) * step < n; i += U * step) {
            v4u qa[U], qb[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                qa[j] = wa[i + j * step];
                qb[j] = DOT ? wb[i + j * step] : qa[j];
            }
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (mine(i + j * step)) reduce_word<P, DOT>(qa[j], qb[j], acc);
        }
        for (; i < n; i += step)
            if (mine(i)) reduce_word<P, DOT>(wa[i], wb[i], acc);
    }
#if LQCD_REDUCE_ATOMIC
    atomicAdd(partial, acc[0]);
    atomicAdd(partial + 1, acc[1]);
#else
    block_sum<2>(acc);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = acc[0];
        partial[2 * blockIdx.x + 1] = acc[1];
    }
#endif
}

// Fixed-order sum of n partial records of two doubles into out[0..1], and (a
// slot given) to the host.
constexpr int FIN_BLOCK = 512;
__global__ __launch_bounds__(FIN_BLOCK) void finalize_k(const double *partial, int64_t n, double *out,
                                                        Mail *mail, uint64_t count) {
    double v[2] = {0.0, 0.0};
    for (int64_t i = threadIdx.x; i < n; i += FIN_BLOCK) {
        v[0] += partial[2 * i];
        v[1] += partial[2 * i + 1];
    }
    block_sum<2>(v);
    if (threadIdx.x == 0) {
        if (mail) {
            mail_post(mail, count, v[0], v[1]);
        } else {
            out[0] = v[0];
            out[1] = v[1];
        }
    }
}

// Kernels of one 16-byte word per thread.
static dim3 word_grid(int64_t n) { return block_grid((n + RED_BLOCK - 1) / RED_BLOCK); }
__device__ __forceinline__ int64_t word_index() { return block_index() * RED_BLOCK + threadIdx.x; }

// y = a x + b y on 16-byte words (FP64, FP32): one word per thread, as the
// copy below (a thread per site: 118 us at 32^4 FP64, full field; now 105, 5.7
// TB/s; FP32 57.4 -> 53.8).
template <typename T>
__global__ __launch_bounds__(RED_BLOCK) void axpby_words_k(T a, const v4u *x, T b, v4u *y, int64_t n) {
    const int64_t i = word_index();
    if (i >= n) return;
    constexpr int R = WORD / (int)sizeof(T);
    T vx[R], vy[R];
    const v4u qx = x[i];
    v4u qy = y[i];
    __builtin_memcpy(vx, &qx, WORD);
    __builtin_memcpy(vy, &qy, WORD);
#pragma unroll
    for (int k = 0; k < R; ++k) vy[k] = fmad(a, vx[k], b * vy[k]);
    __builtin_memcpy(&qy, vy, WORD);
    y[i] = qy;
}

// The same on binary16 fields, site by site for the scale.
__global__ __launch_bounds__(RED_BLOCK) void axpby_f16_k(float a, const char *x, float b, char *y, int64_t vh,
                                                         int nhalf, int64_t hb) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= vh * nhalf) return;
    const int64_t off = s >= vh ? hb : 0;
    if (s >= vh) s -= vh;
    cplx<float> vx[12], vy[12];
    load_spinor<LQCD_F16>(x + off, s, vx);
    load_spinor<LQCD_F16>(y + off, s, vy);
#pragma unroll
    for (int k = 0; k < 12; ++k) vy[k] = {fmad(a, vx[k].re, b * vy[k].re), fmad(a, vx[k].im, b * vy[k].im)};
    store_spinor<LQCD_F16>(y + off, s, vy);
}

template <int PD, int PS>
__global__ __launch_bounds__(RED_BLOCK) void convert_k(char *dst, const char *src, int64_t vh,
                                                       int nhalf, int64_t hbd, int64_t hbs) {
    using TD = typename real_of<PD>::type;
    using TS = typename real_of<PS>::type;
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= vh * nhalf) return;
    const bool hi = s >= vh;
    if (hi) s -= vh;
    cplx<TS> v[12];
    load_spinor<PS>(src + (hi ? hbs : 0), s, v);
    cplx<TD> w[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) w[k] = {(TD)v[k].re, (TD)v[k].im};
    store_spinor<PD>(dst + (hi ? hbd : 0), s, w);
}

// Same storage precision: the layouts agree byte for byte, so the copy is one
// 16-byte word per thread (a thread per site moving all its words measured
// 5.3 TB/s on a 4 GB copy against 6.2 TB/s for one word per thread).
__global__ __launch_bounds__(RED_BLOCK) void copy_words_k(v4u *dst, const v4u *src, int64_t n) {
    const int64_t i = word_index();
    if (i < n) dst[i] = src[i];
}

void launch_convert(const Geom &g, int nhalf, char *dst, int pd, const char *src, int ps,
                    hipStream_t st) {
    if (pd == ps) {
        const int64_t words = (int64_t)half_spinor_bytes(g, pd) * nhalf / 16;
        copy_words_k<<<word_grid(words), RED_BLOCK, 0, st>>>((v4u *)dst, (const v4u *)src, words);
        return;
    }
    const int64_t n = g.vh * nhalf;
    dim3 grid((unsigned)((n + RED_BLOCK - 1) / RED_BLOCK)), block(RED_BLOCK);
    const int64_t hbd = (int64_t)half_spinor_bytes(g, pd), hbs = (int64_t)half_spinor_bytes(g, ps);
#define LQCD_CONV(A, B) \
    if (pd == A && ps == B) { convert_k<A, B><<<grid, block, 0, st>>>(dst, src, g.vh, nhalf, hbd, hbs); return; }
    LQCD_CONV(LQCD_F64, LQCD_F32)
    LQCD_CONV(LQCD_F64, LQCD_F16)
    LQCD_CONV(LQCD_F32, LQCD_F64)
    LQCD_CONV(LQCD_F32, LQCD_F16)
    LQCD_CONV(LQCD_F16, LQCD_F64)
    LQCD_CONV(LQCD_F16, LQCD_F32)
#undef LQCD_CONV
}

void launch_reduce(const Geom &g, int nhalf, const char *a, const char *b, int prec,
                   double *partial, hipStream_t st) {
    const int64_t hb = (int64_t)half_spinor_bytes(g, prec);
    dim3 grid((unsigned)reduce_grid(g, nhalf)), block(RED_BLOCK);
    const bool dot = b != nullptr, ragged = g.vh % TILE != 0;
#define LQCD_RED(P, D, R)                                                                       \
    if (prec == P && dot == D && (ragged == R || P == LQCD_F16)) {                              \
        reduce_k<P, D, R><<<grid, block, 0, st>>>(a, b, g.vh, g.ntiles, nhalf, hb, partial);    \
        return;                                                                                 \
    }
    LQCD_RED(LQCD_F64, false, false)
    LQCD_RED(LQCD_F64, false, true)
    LQCD_RED(LQCD_F64, true, false)
    LQCD_RED(LQCD_F64, true, true)
    LQCD_RED(LQCD_F32, false, false)
    LQCD_RED(LQCD_F32, false, true)
    LQCD_RED(LQCD_F32, true, false)
    LQCD_RED(LQCD_F32, true, true)
    LQCD_RED(LQCD_F16, false, false)
    LQCD_RED(LQCD_F16, true, false)
#undef LQCD_RED
}

}  // namespace lqcd

using namespace lqcd;

static int subset_halves(int subset) {
    return subset == LQCD_FULL ? 2 : (subset == LQCD_EVEN || subset == LQCD_ODD) ? 1 : 0;
}

static bool al16(const void *p) { return p && ((uintptr_t)p & 15) == 0; }

extern "C" size_t lqcd_reduce_workspace_bytes(const lqcd_geom_t *gg, int subset) {
    Geom g;
    const int nh = subset_halves(subset);
    if (!make_geom(gg, &g) || !nh) return 0;
    return (size_t)(2 * reduce_blocks(g, nh) + 2) * sizeof(double);
}

static int reduce_entry(const lqcd_geom_t *gg, int subset, const void *a, const void *b,
                        int prec, void *ws, double *result, void *stream, bool post) {
    Geom g;
    const int nh = subset_halves(subset);
    if (!make_geom(gg, &g) || !nh || !valid_prec(prec)) return LQCD_EINVAL;
    if (!al16(a) || (b && !al16(b)) || !al16(ws) || !result) return LQCD_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    double *partial = (double *)ws;
    double *out = partial + 2 * reduce_blocks(g, nh);
    MailSlot mail;
#if LQCD_REDUCE_ATOMIC
    out = partial;
    hipError_t ez = hipMemsetAsync(out, 0, 2 * sizeof(double), st);
    if (ez != hipSuccess) {
        set_hip_error(ez);
        return LQCD_EHIP;
    }
    launch_reduce(g, nh, (const char *)a, (const char *)b, prec, partial, st);
#else
    launch_reduce(g, nh, (const char *)a, (const char *)b, prec, partial, st);
    if (post) mail.open(st);
    finalize_k<<<1, FIN_BLOCK, 0, st>>>(partial, reduce_grid(g, nh), out, mail.get(),
                                        mail.get() ? mail.next() : 0);
#endif
    int rc = check_launch();
    if (rc) return rc;
    // the stream is synchronised, as the interface says, whichever way the
    // result comes; a posted one saves the copy (|a|^2 at 4^4, whole call: 31
    // -> 20 us; 14 without the synchronisation)
    double host[2];
    if (mail.get()) {
        rc = mail.finish(host, 2);
        if (rc) return rc;
    } else {
        hipError_t e = hipMemcpyAsync(host, out, sizeof(host), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            set_hip_error(e);
            return LQCD_EHIP;
        }
    }
    result[0] = host[0];
    if (b) result[1] = host[1];
    return LQCD_OK;
}

extern "C" int lqcd_dot(const lqcd_geom_t *g, int subset, const void *a, const void *b, int prec,
                        void *workspace, double *result, void *stream) {
    if (!b) return LQCD_EINVAL;
    return reduce_entry(g, subset, a, b, prec, workspace, result, stream, true);
}

// ---------------------------------------------------------------------------
// allocation-free inner product: the block partials live in a static device
// array instead of caller workspace
// ---------------------------------------------------------------------------

// Doubles of the static scratch: two per reduction block plus the two-double
// result, 1 MiB in all (every GPU the library runs on keeps its own copy until
// the process ends).
constexpr int64_t NOALLOC_DOUBLES = (int64_t)1 << 17;
static __device__ __align__(256) double scratch[NOALLOC_DOUBLES];

constexpr int MAX_DEVICES = 64;
static std::mutex scratch_mutex;
static double *scratch_ptr[MAX_DEVICES] = {};

// Device address of this GPU's copy of `scratch`, looked up once per device
// with that device current (the host-side name of the array is not a device
// address and must never reach a kernel).
static int scratch_address(double **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_hip_error(e);
        return LQCD_EHIP;
    }
    if (dev < 0 || dev >= MAX_DEVICES) return LQCD_EINVAL;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol);
            return LQCD_EHIP;
        }
        scratch_ptr[dev] = (double *)p;
    }
    *out = scratch_ptr[dev];
    return LQCD_OK;
}

// two doubles per block of RED_BLOCK sites, plus the result
static_assert((NOALLOC_DOUBLES - 2) / 2 * RED_BLOCK == LQCD_DOT_NOALLOC_MAX_SITES,
              "the header's site limit matches the static scratch");

extern "C" int lqcd_dot_noalloc(const lqcd_geom_t *gg, int subset, const void *a, const void *b,
                                int prec, double *result, void *stream) {
    Geom g;
    const int nh = subset_halves(subset);
    if (!b || !make_geom(gg, &g) || !nh || !valid_prec(prec)) return LQCD_EINVAL;
    if (!al16(a) || !al16(b) || !result) return LQCD_EINVAL;
    const int64_t nb = reduce_blocks(g, nh);
    if (2 * nb + 2 > NOALLOC_DOUBLES) return LQCD_ESMALL;
    double *ws = nullptr;
    const int rc = scratch_address(&ws);
    if (rc) return rc;
    // every partial is written by the reduction before the final sum reads
    // it, so nothing left over from an earlier call needs clearing
    return reduce_entry(gg, subset, a, b, prec, ws, result, stream, false);
}

extern "C" int lqcd_norm2(const lqcd_geom_t *g, int subset, const void *a, int prec,
                          void *workspace, double *result, void *stream) {
    return reduce_entry(g, subset, a, nullptr, prec, workspace, result, stream, true);
}

extern "C" int lqcd_axpby(const lqcd_geom_t *gg, int subset, double a, const void *x, double b,
                          void *y, int prec, void *stream) {
    Geom g;
    const int nh = subset_halves(subset);
    if (!make_geom(gg, &g) || !nh || !valid_prec(prec)) return LQCD_EINVAL;
    if (!al16(x) || !al16(y)) return LQCD_EINVAL;
    const int64_t hb = (int64_t)half_spinor_bytes(g, prec);
    const int64_t n = prec == LQCD_F16 ? g.vh * nh : hb * nh / WORD;
    const dim3 grid = word_grid(n), block(RED_BLOCK);
    hipStream_t st = (hipStream_t)stream;
    if (prec == LQCD_F64) axpby_words_k<double><<<grid, block, 0, st>>>(a, (const v4u *)x, b, (v4u *)y, n);
    else if (prec == LQCD_F32) axpby_words_k<float><<<grid, block, 0, st>>>((float)a, (const v4u *)x, (float)b, (v4u *)y, n);
    else axpby_f16_k<<<grid, block, 0, st>>>((float)a, (const char *)x, (float)b, (char *)y, g.vh, nh, hb);
    return check_launch();
}

extern "C" int lqcd_convert(const lqcd_geom_t *gg, int subset, void *dst, int dst_prec,
                            const void *src, int src_prec, void *stream) {
    Geom g;
    const int nh = subset_halves(subset);
    if (!make_geom(gg, &g) || !nh || !valid_prec(dst_prec) || !valid_prec(src_prec)) return LQCD_EINVAL;
    if (!al16(dst) || !al16(src) || dst == src) return LQCD_EINVAL;
    launch_convert(g, nh, (char *)dst, dst_prec, (const char *)src, src_prec, (hipStream_t)stream);
    return check_launch();
}
