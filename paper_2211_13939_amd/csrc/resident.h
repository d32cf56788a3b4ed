// Which pools of this process may launch beside which.
//
// The workgroups of a segment's launch (segment.hip) wait for each other and take a compute unit each, 24 of the 32 of an XCD (fp32: up to 27), until the
// segment ends.  Two such launches on one device, or one beside another pool's step launches, whose workgroups wait for each other too, could
// each get a part of their workgroups started and wait for the rest until the bound of the waits ends the requests of both.  So on one
// device a segment's launch begins when the other pools' launches so far have ended, and a step's when the other pools' segments have;
// steps of several pools run beside each other (a step's launches leave room for another's workgroups on a compute unit).
//
// The order is the device's: a pool's stream waits for an event on the other's.  An event behind every call is 3.5 to 4.5 us of the queue's time
// (40 steps of one request 378 -> 381 us, each call waited for 393 -> 398), so none is recorded while one thread drives the pools of a device
// and waits for each before it turns to another: a pool whose stream has been waited for has nothing queued, and one that has, gets
// its event when another pool is about to launch.  From the second thread on that drives a pool of the device every call ends with an event:
// a stream's owner may be about to capture it, so nobody else records on it.
// Other processes and launches that a caller has captured are not in these books.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

namespace tts {

enum Gang { GANG_NONE, GANG_STEPS, GANG_SEGMENT };         // launches whose workgroups wait for each other, if any

struct Resident {                                           // a pool in the books of its device
    int device = -1;                                        // -1: not in them
    hipStream_t stream = nullptr;
    hipEvent_t last = nullptr;                              // behind its latest call, where `recorded`
    bool recorded = false;
    std::atomic<int> queued{GANG_NONE};                     // what its stream may still hold
};

struct Neighbours {
    std::mutex m;
    std::vector<Resident*> all;
    std::thread::id thread;                                 // the one thread that has launched so far ...
    bool threads = false;                                   // ... or more than one has
    static Neighbours& of(int device)
    {
        static std::mutex m;
        static std::map<int, Neighbours>* books = new std::map<int, Neighbours>;     // (pools may outlive the statics)
        std::lock_guard<std::mutex> l(m);
        return (*books)[device];
    }
    // Waits for what the others have queued without an event behind it.  A stream that is being captured cannot be waited for.
    void settle(const Resident* but)
    {
        for (Resident* q : all) {
            if (q == but || q->recorded || q->queued == GANG_NONE) continue;
            hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
            if (hipStreamIsCapturing(q->stream, &c) == hipSuccess && c == hipStreamCaptureStatusNone && hipStreamSynchronize(q->stream) == hipSuccess)
                q->queued = GANG_NONE;
            else (void)hipGetLastError();
        }
    }
};

inline hipError_t resident_join(Resident& r, int device, hipStream_t stream)
{
    if (hipError_t e = hipEventCreateWithFlags(&r.last, hipEventDisableTiming)) return e;
    r.device = device;
    r.stream = stream;
    Neighbours& n = Neighbours::of(device);
    std::lock_guard<std::mutex> l(n.m);
    n.settle(&r);                                           // (a pool that was alone has recorded nothing)
    n.all.push_back(&r);
    return hipSuccess;
}

// (the pool's stream has been waited for)
inline void resident_leave(Resident& r)
{
    if (r.device >= 0) {
        Neighbours& n = Neighbours::of(r.device);
        std::lock_guard<std::mutex> l(n.m);
        n.all.erase(std::find(n.all.begin(), n.all.end(), &r));
        if (n.all.empty()) {
            n.threads = false;
            n.thread = std::thread::id();
        }
    }
    if (r.last) (void)hipEventDestroy(r.last);
}

// A call's launches.  Other pools of the device launch before or after all of them.
class Turn {
public:
    Turn(Resident& r, bool captured) : r_(r), n_(Neighbours::of(r.device)), captured_(captured) {}
    Turn(const Turn&) = delete;
    // ahead of a launch of this kind
    hipError_t before(Gang kind)
    {
        if (captured_ || kind <= held_) return hipSuccess;
        if (!lock_.owns_lock()) {
            lock_ = std::unique_lock<std::mutex>(n_.m);
            const std::thread::id me = std::this_thread::get_id();
            if (n_.thread == std::thread::id()) n_.thread = me;
            if (!n_.threads && n_.thread != me) {
                n_.settle(&r_);
                n_.threads = true;
            }
        }
        for (Resident* q : n_.all) {
            if (q->stream == r_.stream || q->queued == GANG_NONE || (kind != GANG_SEGMENT && q->queued != GANG_SEGMENT)) continue;
            if (!n_.threads) {
                hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
                if (hipError_t e = hipStreamIsCapturing(q->stream, &c)) return e;
                if (c != hipStreamCaptureStatusNone) continue;         // (by this thread, which has to have waited for it)
                if (hipStreamQuery(q->stream) == hipSuccess) {
                    q->queued = GANG_NONE;
                    continue;
                }
                (void)hipGetLastError();                               // not ready
                if (hipError_t e = hipEventRecord(q->last, q->stream)) return e;
                if (hipError_t e = hipStreamWaitEvent(r_.stream, q->last, 0)) return e;
            } else if (q->recorded) {
                if (hipError_t e = hipStreamWaitEvent(r_.stream, q->last, 0)) return e;
            }
        }
        held_ = kind;
        return hipSuccess;
    }
    ~Turn()
    {
        if (held_ == GANG_NONE) return;
        r_.queued = std::max<int>(r_.queued, held_);
        const bool alone = std::all_of(n_.all.begin(), n_.all.end(), [&](const Resident* q) { return q->stream == r_.stream; });
        r_.recorded = !alone && n_.threads && hipEventRecord(r_.last, r_.stream) == hipSuccess;
        if (!alone && n_.threads && !r_.recorded) n_.settle(nullptr);
    }

private:
    Resident& r_;
    Neighbours& n_;
    const bool captured_;
    Gang held_ = GANG_NONE;
    std::unique_lock<std::mutex> lock_;
};

}  // namespace tts
