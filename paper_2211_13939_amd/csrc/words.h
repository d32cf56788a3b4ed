// Words through which the workgroups of one launch hand values to each other.  A word is its own flag: a buffer is filled with EMPTY, a
// pattern no value is stored as, and a reader polls until none of its words is EMPTY.
#pragma once
#include "mfma.h"

namespace tts {

constexpr unsigned EMPTY = 0xffffffffu;
// bit of the buffer instructions' cache policy: sc1 = agent scope (loads look past the caches of CU and XCD, stores write through)
constexpr int AGENT = 16;

// this wave's stores so far are acknowledged: stands between the emptying of words and the words of the same step.  Placed where the
// wave has just waited for loads that it requested after the emptying, it costs nothing.
__device__ __forceinline__ void stores_done() { vm_in_flight_at_most<0>(); }

struct Words {
    char* base;
    int bytes, polls;
    // the words of one pool tile
    __device__ __forceinline__ Words of(int tile, int tile_bytes) const { return {base + (size_t)tile * tile_bytes, tile_bytes, polls}; }
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rs() const { return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, BUFFER_RSRC_RAW); }
    // (the compiler may not take a round of polls for the one before)
    __device__ __forceinline__ static void again() { asm volatile("" ::: "memory"); }
    __device__ __forceinline__ u32x4_t look4(int lane_off, int off) const { return __builtin_amdgcn_raw_buffer_load_b128(rs(), lane_off, off, AGENT); }
    __device__ __forceinline__ unsigned look(int lane_off, int off) const { return __builtin_amdgcn_raw_buffer_load_b32(rs(), lane_off, off, AGENT); }
    // EMPTY itself is a NaN with all bits set, as a float and as a pair of halves: stored as another NaN
    __device__ __forceinline__ void put(unsigned v, int lane_off, int off) const
    {
        __builtin_amdgcn_raw_buffer_store_b32(v < EMPTY ? v : EMPTY - 1u, rs(), lane_off, off, AGENT);
    }
    __device__ __forceinline__ void put2(unsigned a, unsigned b, int lane_off, int off) const
    {
        typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{a < EMPTY ? a : EMPTY - 1u, b < EMPTY ? b : EMPTY - 1u}, rs(), lane_off, off, AGENT);
    }
    __device__ __forceinline__ void put4(const floatx4& v, int lane_off, int off) const
    {
        u32x4_t u;
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = __float_as_uint(v[i]) < EMPTY ? __float_as_uint(v[i]) : EMPTY - 1u;
        __builtin_amdgcn_raw_buffer_store_b128(u, rs(), lane_off, off, AGENT);
    }
    __device__ __forceinline__ void empty(int lane_off, int off) const { __builtin_amdgcn_raw_buffer_store_b32(EMPTY, rs(), lane_off, off, AGENT); }
    __device__ __forceinline__ void empty4(int lane_off, int off) const
    {
        __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{EMPTY, EMPTY, EMPTY, EMPTY}, rs(), lane_off, off, AGENT);
    }
    __device__ __forceinline__ static bool full(const u32x4_t& v) { return max(max(v.x, v.y), max(v.z, v.w)) != EMPTY; }

    // Fragments first, first + 8, ... of a B operand (lane = column + 16 * group), STRIDE bytes apart from one to the next, at the
    // lane's offset in a fragment; zeros where the lane's column takes no part.  False: the wait ran out.
    // NAP: pause between polls, in units of 64 cycles (waits that are off the chain)
    template <int N, int STRIDE, int NAP = 0>
    __device__ __forceinline__ bool take(int buf, int first, int lane_off, bool on, uint4 (&out)[N]) const
    {
        u32x4_t w[N];
#pragma unroll
        for (int n = 0; n < N; ++n) w[n] = u32x4_t{0u, 0u, 0u, 0u};
        return take_on<N, STRIDE, NAP>(buf, first, lane_off, !on, w, out);
    }
    // the first look, asked for ahead: loads return in the order of the requests, those behind a store after its acknowledgement
    template <int N, int STRIDE>
    __device__ __forceinline__ void ahead(int buf, int first, int lane_off, u32x4_t (&w)[N]) const
    {
        again();
#pragma unroll
        for (int n = 0; n < N; ++n) w[n] = look4(lane_off, buf + (first + 8 * n) * STRIDE);
    }
    // ... and what is left to be done about it
    template <int N, int STRIDE, int NAP = 0>
    __device__ __forceinline__ bool take_rest(int buf, int first, int lane_off, bool on, u32x4_t (&w)[N], uint4 (&out)[N]) const
    {
        bool in = true;
#pragma unroll
        for (int n = 0; n < N; ++n) {
            in = in && full(w[n]);
            if (!on) w[n] = u32x4_t{0u, 0u, 0u, 0u};
        }
        return take_on<N, STRIDE, NAP>(buf, first, lane_off, in || !on, w, out) && polls > 0;
    }
    template <int N, int STRIDE, int NAP>
    __device__ __forceinline__ bool take_on(int buf, int first, int lane_off, bool in, u32x4_t (&w)[N], uint4 (&out)[N]) const
    {
        for (int spin = 0; spin < polls && !in; ++spin) {
            again();
#pragma unroll
            for (int n = 0; n < N; ++n) w[n] = look4(lane_off, buf + (first + 8 * n) * STRIDE);
            in = true;
#pragma unroll
            for (int n = 0; n < N; ++n) in = in && full(w[n]);
            if constexpr (NAP > 0) {
                if (!in) __builtin_amdgcn_s_sleep(NAP);
            }
        }
#pragma unroll
        for (int n = 0; n < N; ++n) out[n] = make_uint4(w[n].x, w[n].y, w[n].z, w[n].w);
        return in;
    }
};

}  // namespace tts
