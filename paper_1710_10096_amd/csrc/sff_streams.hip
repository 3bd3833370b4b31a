// The library's helper streams, each with a fork and a join event, for calls that
// run two independent launch sequences concurrently (the two fields of a match
// level; the reference and target gradients of the FP32 window cost).  A few per
// device, dealt to the calling threads, so that calls of different threads do not
// queue behind one another.
#include <atomic>

#include "sff_internal.hpp"

namespace sff {
namespace {

constexpr int kMaxHelperDevices = 64, kHelpers = 4;
HelperStream helpers[kMaxHelperDevices][kHelpers];
std::atomic<unsigned> next_thread{0};

bool create(HelperStream& h) {
    hipStream_t s = nullptr;
    hipEvent_t f = nullptr, j = nullptr;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return false;
    if (hipEventCreateWithFlags(&f, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&j, hipEventDisableTiming) != hipSuccess) {
        if (f) (void)hipEventDestroy(f);
        (void)hipStreamDestroy(s);
        return false;
    }
    h.stream = s;
    h.fork = f;
    h.join = j;
    return true;
}

// The capture that st takes part in (0: none); false on an error or a capture that
// has become invalid.  The null stream cannot be captured.
bool capture_of(hipStream_t st, unsigned long long& id) {
    id = 0;
    if (!st) return true;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    unsigned long long c = 0;
    if (hipStreamGetCaptureInfo(st, &status, &c) != hipSuccess) return false;
    if (status == hipStreamCaptureStatusActive) id = c;
    return status != hipStreamCaptureStatusInvalidated;
}

}  // namespace

HelperUse::HelperUse(hipStream_t st) : st_(st) {
    static thread_local const unsigned mine = next_thread++;
    int dev = 0;
    unsigned long long own = 0;
    bool ok = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxHelperDevices && capture_of(st, own);
    for (unsigned k = 0; ok && !h_ && k < kHelpers; ++k) {
        HelperStream& h = helpers[dev][(mine + k) % kHelpers];
        std::unique_lock<std::mutex> lock(h.mutex);
        // created outside captures only; one that takes part in a capture is left to it
        // until that ends
        unsigned long long other = 0;
        if (!h.stream && (own != 0 || !create(h))) continue;
        if (!capture_of(h.stream, other) || (other != 0 && other != own)) continue;
        ok = hipEventRecord(h.fork, st) == hipSuccess && hipStreamWaitEvent(h.stream, h.fork, 0) == hipSuccess;
        if (!ok) break;
        h_ = &h;
        lock_ = std::move(lock);
    }
    if (!h_) (void)hipGetLastError();  // the call goes on without a helper
}

bool HelperUse::join() {
    return hipEventRecord(h_->join, h_->stream) == hipSuccess && hipStreamWaitEvent(st_, h_->join, 0) == hipSuccess;
}

}  // namespace sff
