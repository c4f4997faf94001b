// Numbers for the host without a copy: a kernel writes them into a slot of
// pinned host memory and the host, which has nothing else to do meanwhile,
// watches the slot's count.  An 8-byte copy to pageable memory is a launch of
// its own and a wait for its completion, 20-25 us in which the GPU idles; a
// posted value arrives 2-3 us after the kernel's end.  (A reduction, which
// synchronises its stream in any case, saves the copy alone.)
//
// One 4 KiB page per process, allocated at the first use and kept (64 slots,
// each given out to one call at a time and handed back at its end); a call
// that finds no slot, or no page, copies as before.  The next owner of a slot
// numbers its posts on from the slot's count, so a slot is handed back only
// when every post numbered so far has landed: a call that gives up after a
// launch drains its stream first, and where that fails the slot is retired.
#pragma once

#include "lqcd_internal.h"

namespace lqcd {

struct alignas(64) Mail {
    uint64_t count;  // posts so far: the value of the last one is complete
    double v[2];
};

// A slot for one call and stream, given back at its end; get() is NULL before
// open(), where there is none, and on a stream that is being captured (whose
// kernels do not run: the copy is refused there).
class MailSlot {
public:
    MailSlot() = default;
    ~MailSlot();
    void open(hipStream_t st);
    MailSlot(const MailSlot &) = delete;
    MailSlot &operator=(const MailSlot &) = delete;
    Mail *get() const { return m_; }
    // the number of the next post
    uint64_t next() { return ++n_; }
    // waits for the post numbered last by next(), made by a kernel on the
    // slot's stream: watched for some milliseconds, then by synchronising
    int wait(double *out, int nv);
    // the same, and the stream is synchronised
    int finish(double *out, int nv);

private:
    int take(double *out, int nv) const;

    Mail *m_ = nullptr;
    uint64_t n_ = 0;
    int slot_ = -1;
    hipStream_t st_ = nullptr;
};

// Synchronises the stream, by an event (mail.hip).
hipError_t drain_stream(hipStream_t st);

// One thread of the grid posts v[0..1].
__device__ __forceinline__ void mail_post(Mail *m, uint64_t count, double a, double b) {
    __hip_atomic_store(&m->v[0], a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&m->v[1], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&m->count, count, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace lqcd
