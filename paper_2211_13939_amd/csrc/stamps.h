// How long a call took on the device, from its own launches: the first one stamps the start, every workgroup of the last one its end, with the
// device's steady clock (100 MHz, the same on all XCDs).  A HIP event in front of a call and one behind it cost 7.5 us of the stream's time where
// calls are queued one behind the other; a stamp is a store beside a workgroup's results.  Us a queued call with events -> with stamps (two-byte):
// PostNet of 3 windows 25.6 -> 17.9, of 64 70.5 -> 61.6; a round of the vocoder, 1 window 70.3 -> 63.1, 64 windows 267 -> 260.  Where every call is
// waited for, most of an event's time passes beside the host's: 3 windows 36.9 -> 35.8 us.
#pragma once
#include <hip/hip_runtime.h>

namespace tts {

// Workgroups of the last launch share the end stamps by their number, those of an XCD (dealt by the number's last three bits) a part of them: what
// two of them store to one place is not much apart, and the latest of all is the call's end.  Nothing has to be cleared: the clock only grows.
// Behind them lies the number of the call that they are of: a call that was only captured has none of its own yet.
constexpr int STAMP_ENDS = 256, STAMP_CALL = 1 + STAMP_ENDS, STAMP_BYTES = (STAMP_CALL + 1) * 8;

struct Stamps {
    unsigned long long* at;      // [0] the call's start, [1 ..] ends, [STAMP_CALL] its number; null: the call is not timed
    unsigned long long call;     // ... from 1 on
#ifdef __HIPCC__
    // The start is read first and stored last: a store ahead of a wave's loads would hold them up until it is acknowledged.
    __device__ __forceinline__ unsigned long long now() const { return at ? wall_clock64() : 0; }
    __device__ __forceinline__ void begin(unsigned long long when) const
    {
        if (at && (blockIdx.x | blockIdx.y | blockIdx.z | threadIdx.x) == 0) {
            at[0] = when;
            at[STAMP_CALL] = call;
        }
    }
    // by a thread of the workgroup that is through
    __device__ __forceinline__ void end() const
    {
        const unsigned wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
        if (at) at[1 + (wg & 7) * (STAMP_ENDS / 8) + (wg >> 3) % (STAMP_ENDS / 8)] = wall_clock64();
    }
#endif
};

}  // namespace tts
