// The attention's location features for one tile of 16 positions, as matrix products whose constant operands a wave holds in
// registers: shared by the attention kernel of the step and the kernel that runs a whole segment of steps.  Device code only.
#pragma once
#include "dev.h"
#include "mfma.h"

namespace tts {

template <typename XT> struct LsaTile;

// fp32: v_mfma_f32_16x16x4_f32, lane group g supplies k = g of each 4-wide step
template <> struct LsaTile<float> {
    float kA[2][16];   // [mt][c*8+s]: filter 16 mt + jl, tap 4 s + g of channel c
    float4 wA[8][2];   // [at][mt]: W_loc row 32 (jl/4) + 4 at + jl%4, filters 16 mt + 4 g .. +3
    __device__ __forceinline__ void load(const DevPtrs& d, int lane)
    {
        const float* kf = reinterpret_cast<const float*>(d.lsa_kfrag);
        const float4* wf = reinterpret_cast<const float4*>(d.lsa_wfrag);
#pragma unroll
        for (int i = 0; i < 32; ++i) kA[i >> 4][i & 15] = kf[i * 64 + lane];
#pragma unroll
        for (int i = 0; i < 16; ++i) wA[i >> 1][i & 1] = wf[i * 64 + lane];
    }
    // x0 = index into s_u of this lane's position at tap 0
    // pl[at] = q[at] + W_loc loc: the query rides in as the accumulator's start value
    __device__ __forceinline__ void run(const float* u0, const float* u1, int x0, int g, const floatx4* q, floatx4* pl) const
    {
        floatx4 loc0 = {0.f, 0.f, 0.f, 0.f}, loc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cs = 0; cs < 16; ++cs) {
            const float b = (cs < 8 ? u0 : u1)[x0 + g + 4 * (cs & 7)];
            loc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kA[0][cs], b, loc0, 0, 0, 0);
            loc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kA[1][cs], b, loc1, 0, 0, 0);
        }
#pragma unroll
        for (int at = 0; at < 8; ++at) {
            floatx4 p = q[at];
            p = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[at][0].x, loc0[0], p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[at][0].y, loc0[1], p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[at][0].z, loc0[2], p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[at][0].w, loc0[3], p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[at][1].x, loc1[0], p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[at][1].y, loc1[1], p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[at][1].z, loc1[2], p, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_16x16x4f32(wA[at][1].w, loc1[3], p, 0, 0, 0);
            pl[at] = p;
        }
    }
};

// two-byte operands: v_mfma_f32_16x16x32_f16, lane group g supplies 8 k values per step
template <> struct LsaTile<h16_t> {
    uint4 kA[2][2];    // [mt][c]: filter 16 mt + jl, taps 8 g .. 8 g + 7 of channel c
    uint4 wA[8];       // [at]: W_loc row 32 (jl/4) + 4 at + jl%4, filters {4g..4g+3, 16+4g..16+4g+3}
    static constexpr int LDS_VECS = 12 * 64;   // the operands of all 64 lanes, as 16-byte pieces
    // the operands are the same for every wave: the workgroup fetches them once into LDS ...
    __device__ static __forceinline__ uint4 fetch(const DevPtrs& d, int i)
    {
        const uint4* kf = reinterpret_cast<const uint4*>(d.lsa_kfrag);
        const uint4* wf = reinterpret_cast<const uint4*>(d.lsa_wfrag);
        return i < 4 * 64 ? kf[i] : wf[i - 4 * 64];
    }
    // ... and every wave takes its lanes' share from there
    __device__ __forceinline__ void load(const uint4* lds, int lane)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) kA[i >> 1][i & 1] = lds[i * 64 + lane];
#pragma unroll
        for (int i = 0; i < 8; ++i) wA[i] = lds[(4 + i) * 64 + lane];
    }
    // loc^T of the tile as the second product's B operand (it does not depend on the query)
    __device__ __forceinline__ uint4 loc(const float* u0, const float* u1, int x0, int g) const
    {
        floatx4 loc0 = {0.f, 0.f, 0.f, 0.f}, loc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float* u = (c == 0 ? u0 : u1) + x0 + 8 * g;
            uint4 b;
            b.x = pack2<h16_t>(u[0], u[1]); b.y = pack2<h16_t>(u[2], u[3]);
            b.z = pack2<h16_t>(u[4], u[5]); b.w = pack2<h16_t>(u[6], u[7]);
            loc0 = mfma_frag<h16_t>(kA[0][c], b, loc0);
            loc1 = mfma_frag<h16_t>(kA[1][c], b, loc1);
        }
        uint4 bl;
        bl.x = pack2<h16_t>(loc0[0], loc0[1]); bl.y = pack2<h16_t>(loc0[2], loc0[3]);
        bl.z = pack2<h16_t>(loc1[0], loc1[1]); bl.w = pack2<h16_t>(loc1[2], loc1[3]);
        return bl;
    }
    __device__ __forceinline__ void run(const float* u0, const float* u1, int x0, int g, const floatx4* q, floatx4* pl) const
    {
        const uint4 bl = loc(u0, u1, x0, g);
#pragma unroll
        for (int at = 0; at < 8; ++at) pl[at] = mfma_frag<h16_t>(wA[at], bl, q[at]);
    }
};

}  // namespace tts
