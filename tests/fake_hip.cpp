// A HIP runtime and the kernels' launch wrappers on host memory, for the host side of the library alone: streams run what is
// queued at once, except that what a kernel still has to read of pinned memory counts as pending until the host has waited for
// it.  Any call can be made to fail (fake_fail), and a slot can be frozen as a kernel would that gave up (fake_freeze).
// A fill of device memory at creation counts as under way until the host has waited (fake_filling).
// What is ordered behind what is followed through streams, events and the host's waits: a segment of steps that is not ordered against another
// stream's steps, or the other way round, counts (fake_unordered).
// A segment's workgroups may start late: what they go by is looked at before the segment and again behind each of its steps, and must be the same,
// and right, for every request that was not lost on the way (fake_stale).
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "../paper_2211_13939_amd/csrc/encoder_kernels.h"
#include "../paper_2211_13939_amd/csrc/kernels.h"
#include "../paper_2211_13939_amd/csrc/vocoder_kernels.h"

namespace {

struct Fail { int in, times; };
std::map<std::string, int> calls;               // calls so far
std::map<std::string, Fail> fails;              // the call that fails, counted from the time of fake_fail, and how many from there on
struct Pending { const void* at; int seq; };
std::vector<Pending> pending;                   // pinned memory that queued work still reads
int seq = 0, violations = 0;                    // violations: such memory rewritten or freed
int freeze_slot = -1, freeze_at = 0;

using Clock = std::map<hipStream_t, int>;       // how much of every stream's work lies before
struct Event { int seq = 0; Clock clock; };
struct Launched { hipStream_t stream; int at; bool segment; };
std::mutex order;
std::map<hipStream_t, Clock> streams;
std::vector<Launched> launched;
int unordered = 0, segments = 0, stale = 0;
bool filling = false;
bool busy = false;                              // what hipStreamQuery says
hipStream_t capturing = nullptr;
Clock host;                                     // what some thread has waited for has ended
void merge(Clock& a, const Clock& b)
{
    for (const auto& kv : b) a[kv.first] = std::max(a[kv.first], kv.second);
}
void ordered(hipStream_t s, bool segment)
{
    std::lock_guard<std::mutex> l(order);
    Clock& c = streams[s];
    merge(c, host);
    for (const Launched& x : launched)
        unordered += x.stream != s && (segment || x.segment) && c[x.stream] < x.at;
    launched.push_back({s, ++c[s], segment});
    segments += segment;
}
void waited(hipStream_t s)
{
    std::lock_guard<std::mutex> l(order);
    merge(host, streams[s]);
}

std::mutex book;
hipError_t call(const char* what)
{
    std::lock_guard<std::mutex> l(book);
    ++calls[what];
    auto it = fails.find(what);
    if (it == fails.end() || --it->second.in > 0) return hipSuccess;
    if (--it->second.times <= 0) fails.erase(it);
    return hipErrorUnknown;
}
void done_up_to(int s)
{
    std::lock_guard<std::mutex> l(book);
    pending.erase(std::remove_if(pending.begin(), pending.end(), [&](const Pending& p) { return p.seq <= s; }), pending.end());
}
bool is_pending(const void* at)
{
    return std::any_of(pending.begin(), pending.end(), [&](const Pending& p) { return p.at == at; });
}

}  // namespace

extern "C" {
void fake_fail(const char* what, int nth, int times) { fails[what] = {nth, times}; }
void fake_reset()
{
    fails.clear();
    freeze_slot = -1;
    pending.clear();
    streams.clear();
    launched.clear();
    violations = unordered = segments = stale = 0;
    busy = filling = false;
    capturing = nullptr;
}
int fake_filling() { return filling; }
void fake_busy(int on) { busy = on; }
void fake_capture(void* stream) { capturing = (hipStream_t)stream; }
int fake_unordered() { return unordered; }
int fake_segments() { return segments; }
int fake_stale() { return stale; }
int fake_calls(const char* what) { return calls[what]; }
int fake_violations() { return violations; }
void fake_freeze(int slot, int at_frame) { freeze_slot = slot; freeze_at = at_frame; }

hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*)
{
    memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize()
{
    filling = false;
    done_up_to(seq);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    if (hipError_t e = call("hipHostMalloc")) return e;
    *p = malloc(n);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipHostFree(void* p)
{
    violations += is_pending(p);
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n)
{
    filling = true;
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    if (hipError_t e = call("hipMemcpyAsync")) return e;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    if (hipError_t e = call("hipStreamSynchronize")) return e;
    filling = filling && s;
    done_up_to(seq);
    waited(s);
    return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s)
{
    if (busy) return hipErrorNotReady;
    waited(s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    if (hipError_t x = call("hipStreamWaitEvent")) return x;
    std::lock_guard<std::mutex> l(order);
    merge(streams[s], reinterpret_cast<Event*>(e)->clock);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c)
{
    *c = s && s == capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new Event); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(new Event); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<Event*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    if (hipError_t x = call("hipEventRecord")) return x;
    std::lock_guard<std::mutex> l(order);
    reinterpret_cast<Event*>(e)->seq = seq;
    reinterpret_cast<Event*>(e)->clock = streams[s];
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { done_up_to(reinterpret_cast<Event*>(e)->seq); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

namespace tts {

hipError_t launch_encoder(const EncoderPtrs&, int, const PnWindows&, int, const EncStaged& staged, float*, hipStream_t)
{
    violations += is_pending(staged.ids);       // the host has written the ids by now
    pending.push_back({staged.ids, ++seq});     // the first kernel is queued whether or not a later launch fails
    return call("launch_encoder");
}

hipError_t launch_postnet_pack(const PostnetPtrs&, int, const PnWindows&, const float*, int, int, bool, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_postnet_chain(const PostnetPtrs&, int, const PnWindows&, const float*, int, float*, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_postnet(const PostnetPtrs&, int, const float*, int, float*, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_vocoder(const VocoderPtrs&, int, const VocBatch&, const float*, float*, hipStream_t) { return hipErrorNotSupported; }

// frame f of a request of n frames: all of its values are 1000 n + f
hipError_t launch_step(const DevPtrs& d, const StepLaunch& cfg, int, hipStream_t stream, hipEvent_t*)
{
    ordered(stream, cfg.seg_steps > 0);
    std::vector<int> left(cfg.seg_steps > 0 ? cfg.n_blocks : 0);
    for (int s = 0; s < (int)left.size(); ++s) left[s] = d.live[s] && !d.done[s] ? d.n_steps[s] - d.t[s] : 0;
    auto look = [&] {
        for (int s = 0; s < (int)left.size(); ++s) stale += !d.failed[s] && segment_left(d, cfg.seg_left, s) != left[s];
    };
    look();
    for (int k = 0; k < std::max(cfg.seg_steps, 1); ++k) {
        for (int s = 0; s < cfg.n_blocks; ++s) {
            if (!d.live[s] || d.done[s]) continue;
            if (s == freeze_slot && d.t[s] >= freeze_at) {
                d.failed[s] = d.done[s] = 1;
                *d.fault = 1;
                continue;
            }
            std::fill_n(d.mel_ring + ((size_t)s * d.max_steps + d.t[s]) * N_MEL, N_MEL, 1000.f * d.n_steps[s] + d.t[s]);
            if (++d.t[s] >= d.n_steps[s]) d.done[s] = 1;
        }
        look();
    }
    return hipSuccess;
}
hipError_t launch_set_live(const DevPtrs& d, const LiveArgs& a, hipStream_t)
{
    for (int s = 0; s < MAX_POOL; ++s) d.live[s] = a.bits[s >> 5] >> (s & 31) & 1;
    return hipSuccess;
}
hipError_t launch_join(const DevPtrs& d, int, int, const JoinArgs& ja, int n, hipStream_t)
{
    for (int i = 0; i < n; ++i) {
        const int s = ja.slot[i];
        d.L[s] = ja.L[i];
        d.n_steps[s] = ja.n_steps[i];
        d.t[s] = d.done[s] = d.failed[s] = 0;
        std::fill_n(d.mel_ring + (size_t)s * d.max_steps * N_MEL, (size_t)d.max_steps * N_MEL, -1.f);   // frames never made
    }
    return hipSuccess;
}
hipError_t launch_stage_chunks(const DevPtrs& d, const StageArgs& sa, int n, int, float* dst, hipStream_t)
{
    if (hipError_t e = call("launch_stage_chunks")) return e;
    for (int i = 0; i < n; ++i)
        memcpy(dst + (size_t)sa.to[i] * N_MEL, d.mel_ring + (size_t)sa.row[i] * N_MEL, (size_t)sa.frames[i] * N_MEL * 4);
    return hipSuccess;
}
hipError_t launch_move_slots(const DevPtrs& d, int, int, const MoveArgs& mv, int n, hipStream_t)
{
    for (int i = 0; i < n; ++i) {
        const int from = mv.from[i], to = mv.to[i];
        for (int* a : {d.L, d.t, d.n_steps, d.done, d.failed}) a[to] = a[from];
        d.failed[from] = 0;
        std::copy_n(d.mel_ring + (size_t)from * d.max_steps * N_MEL, (size_t)d.max_steps * N_MEL, d.mel_ring + (size_t)to * d.max_steps * N_MEL);
    }
    return hipSuccess;
}
hipError_t launch_presum_tile(const DevPtrs&, int, int, int, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_prenet_slot(const DevPtrs&, int, int, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_x_get(int, const void*, int, int, int, int, float*, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_x_set(int, void*, int, int, int, int, const float*, hipStream_t) { return hipErrorNotSupported; }

}  // namespace tts
