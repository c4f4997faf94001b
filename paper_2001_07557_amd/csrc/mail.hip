// Slots of pinned host memory that kernels post numbers into (mail.h).

#include <chrono>
#include <mutex>

#include "mail.h"

namespace lqcd {

// (0, for a test build: every call copies its numbers)
#ifndef LQCD_MAIL_SLOTS
#define LQCD_MAIL_SLOTS 64
#endif
constexpr int MAIL_SLOTS = LQCD_MAIL_SLOTS;
static std::mutex mail_mutex;
static Mail *mail_page = nullptr;
static uint64_t mail_used = 0;  // a bit per slot
static_assert(MAIL_SLOTS <= 64 && MAIL_SLOTS * sizeof(Mail) <= 4096, "one page, a bit per slot");

void MailSlot::open(hipStream_t st) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    if (status != hipStreamCaptureStatusNone || MAIL_SLOTS == 0) return;
    std::lock_guard<std::mutex> lock(mail_mutex);
    if (!mail_page) {
        // (allowed while another thread captures a graph)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        void *p = nullptr;
        const hipError_t e = hipHostMalloc(&p, MAIL_SLOTS * sizeof(Mail),
                                           hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent);
        if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        mail_page = static_cast<Mail *>(p);
    }
    for (int i = 0; i < MAIL_SLOTS; ++i)
        if (!((mail_used >> i) & 1)) {
            mail_used |= (uint64_t)1 << i;
            slot_ = i;
            st_ = st;
            m_ = mail_page + i;
            n_ = __atomic_load_n(&m_->count, __ATOMIC_ACQUIRE);
            return;
        }
}

MailSlot::~MailSlot() {
    if (slot_ < 0) return;
    // a post that is still to come would carry the number of the next owner's
    // first (a launch that failed never posts: its number is not reached, and
    // nothing is pending once the stream has drained)
    if (__atomic_load_n(&m_->count, __ATOMIC_ACQUIRE) != n_ && hipStreamSynchronize(st_) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    std::lock_guard<std::mutex> lock(mail_mutex);
    mail_used &= ~((uint64_t)1 << slot_);
}

// The host watches a slot this long before it lets the runtime wait, which
// frees the core and wakes up some 20 us late: ten iterations of a solve, the
// time between its reads, are 0.3 ms at 16^4 (FP32) and 1.3 ms at 32^4
// (binary16); what else the caller has queued may take any time.
constexpr std::chrono::milliseconds WATCH(4);

int MailSlot::wait(double *out, int nv) {
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t spin = 1; __atomic_load_n(&m_->count, __ATOMIC_ACQUIRE) != n_; ++spin) {
        __builtin_ia32_pause();
        if (spin % 1024 == 0 && std::chrono::steady_clock::now() - t0 > WATCH) {
            const hipError_t e = hipStreamSynchronize(st_);
            if (e != hipSuccess) {
                set_hip_error(e);
                return LQCD_EHIP;
            }
            break;  // (a drained stream that posted nothing is take's error)
        }
    }
    return take(out, nv);
}

// An event behind the post is waited for in the stream's place: once five or
// six launches have gone before it, hipStreamSynchronize returns 30 us after
// the last one has ended, an event 6 us after (a reduction behind eight shifts
// of 8^4, whole sequence: 83 -> 53 us; 48-54 without either; at the end of a
// solve, hundreds of launches, 24^3x48 FP32 with force 8586 -> 8494 us).
int MailSlot::finish(double *out, int nv) {
    hipEvent_t ev;
    const bool have = hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess;
    const bool recorded = have && hipEventRecord(ev, st_) == hipSuccess;
    if (!recorded) (void)hipGetLastError();
    const int rc = wait(out, nv);
    hipError_t e = hipSuccess;
    if (!rc) e = recorded ? hipEventSynchronize(ev) : hipStreamSynchronize(st_);
    if (have) (void)hipEventDestroy(ev);
    if (e != hipSuccess) {
        set_hip_error(e);
        return LQCD_EHIP;
    }
    return rc;
}

hipError_t drain_stream(hipStream_t st) {
    hipEvent_t ev;
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        return hipStreamSynchronize(st);
    }
    hipError_t e = hipEventRecord(ev, st);
    if (e == hipSuccess) {
        e = hipEventSynchronize(ev);
    } else {
        (void)hipGetLastError();
        e = hipStreamSynchronize(st);
    }
    (void)hipEventDestroy(ev);
    return e;
}

int MailSlot::take(double *out, int nv) const {
    if (__atomic_load_n(&m_->count, __ATOMIC_ACQUIRE) != n_) {
        set_hip_error(hipErrorUnknown);
        return LQCD_EHIP;
    }
    for (int i = 0; i < nv; ++i) __atomic_load(&m_->v[i], &out[i], __ATOMIC_RELAXED);
    return LQCD_OK;
}

}  // namespace lqcd
