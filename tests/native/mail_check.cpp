// Host check of the slots through which kernels post numbers (csrc/mail.hip),
// with the few HIP calls it makes replaced by a stream that is played by hand:
// posts are queued and land when the stream is drained, or when told to.
// Prints one line per check and "checks N bad B".
#include <string.h>

#include "mail.hip"

#include <cstdio>
#include <cstdlib>
#include <ctime>
#include <deque>

namespace {

struct Post {
    lqcd::Mail *m;
    uint64_t count;
    double v[2];
};
std::deque<Post> queue;   // enqueued, not yet run
bool drain_fails = false, record_fails = false;
int drains = 0, events = 0;

void enqueue(lqcd::MailSlot &s, double a, double b) { queue.push_back({s.get(), s.next(), {a, b}}); }
void run_all() {
    for (; !queue.empty(); queue.pop_front()) {
        const Post &p = queue.front();
        p.m->v[0] = p.v[0];
        p.m->v[1] = p.v[1];
        __atomic_store_n(&p.m->count, p.count, __ATOMIC_RELEASE);
    }
}

int checks = 0, bad = 0;
void check(bool ok, const char *what) {
    ++checks;
    bad += !ok;
    printf("%s %s\n", ok ? "ok  " : "FAIL", what);
}

}  // namespace

extern "C" {
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = aligned_alloc(4096, n);
    ::memset(*p, 0, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    ++drains;
    if (drain_fails) return hipErrorUnknown;
    run_all();
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return record_fails ? hipErrorUnknown : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
    ++events;
    return hipStreamSynchronize(nullptr);
}
hipError_t hipGetLastError(void) { return hipSuccess; }
}

namespace lqcd {
void set_hip_error(hipError_t) {}
}

using namespace lqcd;

int main() {
    setvbuf(stdout, nullptr, _IONBF, 0);
    // a call that gives up after its launch: the next one must not take its number
    {
        Mail *first;
        {
            MailSlot a;
            a.open(nullptr);
            first = a.get();
            enqueue(a, 1.0, -1.0);
        }
        check(queue.empty() || drains > 0, "an abandoned post is waited for");
        MailSlot b;
        b.open(nullptr);
        const uint64_t before = __atomic_load_n(&b.get()->count, __ATOMIC_ACQUIRE);
        const uint64_t n = b.next();
        run_all();
        check(b.get() != first || __atomic_load_n(&first->count, __ATOMIC_ACQUIRE) != n,
              "a late post does not carry the next owner's number");
        check(b.get()->count == before, "no post lands in the slot of another call");
    }
    // the same where the stream cannot be drained: the slot is never given out again
    {
        Mail *lost;
        {
            MailSlot a;
            a.open(nullptr);
            lost = a.get();
            enqueue(a, 2.0, -2.0);
            drain_fails = true;
        }
        drain_fails = false;
        MailSlot b;
        b.open(nullptr);
        check(b.get() && b.get() != lost, "a slot whose post may still come is retired");
        run_all();
    }
    // a post that does not come while the host watches: it stops watching and
    // lets the runtime wait
    {
        MailSlot a;
        a.open(nullptr);
        enqueue(a, 3.0, 4.0);
        double out[2] = {0, 0};
        const int was = drains;
        const clock_t t0 = clock();
        const int rc = a.wait(out, 2);
        const double cpu = (double)(clock() - t0) / CLOCKS_PER_SEC;
        check(rc == LQCD_OK && out[0] == 3.0 && out[1] == 4.0, "a late post is received");
        check(drains > was && cpu < 1.0, "the host stops watching after a while");
    }
    // a result that is waited for together with its stream, by an event or
    // without one
    for (bool fails : {false, true}) {
        record_fails = fails;
        MailSlot a;
        a.open(nullptr);
        enqueue(a, 7.0, 8.0);
        run_all();
        double out[2];
        const int was = drains, ev = events;
        check(a.finish(out, 2) == LQCD_OK && out[0] == 7.0 && out[1] == 8.0 && drains > was &&
                  events == ev + !fails,
              "a finished call has drained its stream");
        record_fails = false;
    }
    for (bool fails : {false, true}) {
        record_fails = fails;
        const int was = drains, ev = events;
        check(drain_stream(nullptr) == hipSuccess && drains == was + 1 && events == ev + !fails,
              "a stream is drained, by an event or without one");
        record_fails = false;
    }
    // a stream that fails, and one that ends without a post
    {
        MailSlot a;
        a.open(nullptr);
        enqueue(a, 5.0, 6.0);
        drain_fails = true;
        double out[2];
        check(a.wait(out, 2) == LQCD_EHIP, "a stream error is returned");
        drain_fails = false;
        run_all();
        MailSlot b;
        b.open(nullptr);
        b.next();
        check(b.wait(out, 2) == LQCD_EHIP, "a post that never comes is an error");
    }
    // slots run out, come back, and the numbers of a slot go on
    {
        MailSlot many[80];
        int got = 0;
        for (auto &s : many) {
            s.open(nullptr);
            got += s.get() != nullptr;
        }
        check(got < 80 && got >= 60, "a call that finds no slot gets none");
    }
    {
        MailSlot a;
        a.open(nullptr);
        double out[2];
        bool ok = a.get() != nullptr;
        for (int i = 0; i < 5 && ok; ++i) {
            enqueue(a, i, i + 0.5);
            run_all();
            ok = a.wait(out, 2) == LQCD_OK && out[0] == i && out[1] == i + 0.5;
        }
        check(ok, "posts of one call arrive in order");
    }
    printf("checks %d bad %d\n", checks, bad);
    return bad ? 1 : 0;
}
