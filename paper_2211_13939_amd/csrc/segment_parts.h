// What the workgroups of a segment of decoder steps have in common, whatever the weights are stored as (segment.hip, segment32.hip).
// Device code only.
#pragma once
#include "dev.h"
#include "mfma.h"
#include "words.h"

namespace tts {
namespace {

constexpr int NT = 512, NW = 8;                             // a workgroup
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

// x of the lane 16 or 32 away, and of the lanes of a row of 16 at a distance: the sums below add the same pairs as the
// step's kernels do with shuffles, without a trip through LDS each
__device__ __forceinline__ float xor16(float v)
{
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(threadIdx.x & 16 ? sw[0] : sw[1]);
}
__device__ __forceinline__ float xor32(float v)
{
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(threadIdx.x & 32 ? sw[0] : sw[1]);
}
template <int N> __device__ __forceinline__ float ror16(float v)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float wave_sum_fast(float v)
{
    v += xor32(v);
    v += xor16(v);
    v += ror16<8>(v);      // from here on a row's values repeat every eight, four, two lanes: a rotation meets the lane an xor would
    v += ror16<4>(v);
    v += ror16<2>(v);
    v += ror16<1>(v);
    return v;
}

// operands that do not change from step to step stay as they are loaded: without this the compiler keeps their conversions, twice
// the registers, outside of the loop over the steps
__device__ __forceinline__ void keep(u32x4_t& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ uint4 as_uint4(const u32x4_t& v) { return make_uint4(v.x, v.y, v.z, v.w); }

__device__ __forceinline__ void cell(const floatx4& g, float& c, float& h)
{
    const float gi = sigmoidf_(g[0]), gf = sigmoidf_(g[1]);
    const float gg = tanhf_(g[2]), go = sigmoidf_(g[3]);
    c = gf * c + gi * gg;
    h = go * tanhf_(c);
}

// What a workgroup knows of the requests: the steps each slot still has to take, from the segment's first on (0: no request there).
struct Pool {
    int cur, n_steps, n_tiles, tile_bytes;
    const int* rem;                                         // [n_tiles * 16], in LDS
};
// the requests that take part in step s end here
__device__ __forceinline__ void give_up(const DevPtrs& d, const Pool& pl, int s)
{
    if ((int)threadIdx.x < pl.n_tiles * 16 && s < pl.rem[threadIdx.x]) {
        d.done[threadIdx.x] = 1;
        d.failed[threadIdx.x] = 1;
        *d.fault = 1;
    }
}

__device__ __forceinline__ void lose_one(const DevPtrs& d, int slot)
{
    if (threadIdx.x == 0) {
        d.done[slot] = 1;
        d.failed[slot] = 1;
        *d.fault = 1;
    }
}

// A barrier at which the waves also learn whether one of them gave up waiting.  `failed` holds the first phase in which one did
// and phases only grow, so a wave that is late to look does not see the failure of a later phase.
struct Phases {
    int* failed;
    int ph = 0;
    __device__ __forceinline__ void sync(bool ok)
    {
        if (!ok) atomicMin(failed, ph);
        lds_barrier();
        ++ph;
    }
    __device__ __forceinline__ bool bad() const { return *failed < ph; }
};

__device__ __forceinline__ int next3(int b) { return b == 2 ? 0 : b + 1; }

}  // namespace
}  // namespace tts
