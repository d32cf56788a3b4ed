// Acoustic encoder kernels (Sec. 2.1.2, Eq. 1) for a ragged batch of requests whose tokens are packed back to back:
//   k_enc_embed   E_all = sum of the four embedding rows of every token, stored as the first convolution's input
//   (conv5_kernels.h: three kernel-5 convolutions with ReLU, "same" padding inside each request)
//   k_enc_xproj   W_ih x + b for every token and both directions: the part of the LSTM that has no recurrence
//   the recurrence, a chain of L dependent steps of a 1024 x 256 matrix-vector product (latency, not bandwidth):
//   k_enc_lstm_sp      two-byte weights, one workgroup per direction and request, the matrix resident in its CU
//   k_enc_lstm_shared  fp32 weights, several workgroups per direction and request(s), the matrix spread over their registers
//   k_enc_lstm_alone   fp32 weights, one workgroup per direction and request: where the former's workgroups did not all start
// The gate rows of W_ih, the biases and the fp32 W_hh are stored unit-major / gate-minor, so the four gate sums of a unit
// are contiguous; the two-byte W_hh has one gate of 16 units per row tile.
#include "encoder_kernels.h"

#include "conv5_chain.h"

namespace tts {
namespace {

struct EncTables { const float* t[ENC_TABLES]; };

// One wave per column, eight channels a lane.  The ids and the per-column table of the convolutions (staged.meta: request
// length << 16 | position inside the request) come straight from the call's pinned staging buffer: one trip over the host link
// in place of four copies and a kernel that expanded the table.  The words through which k_enc_lstm_shared's workgroups
// exchange h, and the one that says that it gave up, are cleared here as well (n_words; none in the two-byte mode).
template <typename XT>
__global__ __launch_bounds__(256) void k_enc_embed(EncTables tb, EncStaged staged, int n_col, int n_col_pad, XT* __restrict__ X,
                                                   int* __restrict__ cmeta, uint32_t* __restrict__ hx, int n_words, int* __restrict__ gave_up)
{
    constexpr int KB = Frag<XT>::KB, EPL = Frag<XT>::EPL;
    const int col = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n_words; i += gridDim.x * 256) hx[i] = 0;
    if (n_words > 0 && blockIdx.x == 0 && threadIdx.x == 0) *gave_up = 0;
    if (col >= n_col_pad) return;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int meta = 0;
    if (col < n_col) {
        const int4 id = staged.ids[col];
        meta = staged.meta[col];
        const int row[ENC_TABLES] = {id.x, id.y, id.z, id.w};
#pragma unroll
        for (int t = 0; t < ENC_TABLES; ++t) {
            const float4* e = reinterpret_cast<const float4*>(tb.t[t] + (size_t)row[t] * ENC_DIM) + 2 * lane;
            const float4 lo = e[0], hi = e[1];
            v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
            v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
        }
    }
#pragma unroll
    for (int i = 0; i < 8; i += EPL) {
        XT* dst = X + xoff<XT>(ENC_DIM / KB, col, 8 * lane + i);
        if constexpr (sizeof(XT) == 2) *reinterpret_cast<uint4*>(dst) = make_uint4(pack2<XT>(v[0], v[1]), pack2<XT>(v[2], v[3]), pack2<XT>(v[4], v[5]), pack2<XT>(v[6], v[7]));
        else *reinterpret_cast<float4*>(dst) = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
    }
    if (lane == 0) cmeta[col] = meta;
}

// grid = (row tiles / 4, column tiles, 2 directions); a wave = one 16-row tile x one 16-column tile, K = dim
template <typename XT>
__global__ __launch_bounds__(256) void k_enc_xproj(const uint4* __restrict__ W0, const uint4* __restrict__ W1, const float* __restrict__ b0,
                                                   const float* __restrict__ b1, const uint4* __restrict__ X, int n_col, int max_tokens,
                                                   float* __restrict__ Y)
{
    constexpr int NKF = ENC_DIM / Frag<XT>::KB;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int rt = blockIdx.x * 4 + wave, ct = blockIdx.y, dir = blockIdx.z;
    const uint4* W = dir ? W1 : W0;
    const float* b = dir ? b1 : b0;
    floatx4 acc = *reinterpret_cast<const floatx4*>(b + rt * 16 + 4 * g);
#pragma unroll 4
    for (int kf = 0; kf < NKF; ++kf) acc = mfma_frag<XT>(W[xfrag(NKF, rt, kf, lane)], X[xfrag(NKF, ct, kf, lane)], acc);
    const int col = ct * 16 + n;
    if (col < n_col) *reinterpret_cast<floatx4*>(Y + ((size_t)dir * max_tokens + col) * ENC_GATES + rt * 16 + 4 * g) = acc;
}

// The three convolutions and the input projection of a small call as one launch (conv5_chain.h).  A workgroup's share of the projection
// are four row tiles, two waves each; every sum is the one chain over k that it is above.
template <typename XT> struct EncChain {
    static constexpr bool TIMED = false;
    static constexpr int LAYERS = ENC_CONVS, CIN = ENC_DIM, EPI = PN_EPI_RELU, EPL = Frag<XT>::EPL, KB = Frag<XT>::KB, NKF = ENC_DIM / KB, LAST = NKF;
    static constexpr int WG_RTS = 2 * ENC_GATES / 16 / CHAIN_RTS, PER = PN_WAVES / WG_RTS;
    const uint4* X;
    const int* cmeta;
    int n_col, max_tokens;
    const uint4 *W0, *W1;
    const float *b0, *b1;
    float* Y;
    __device__ __forceinline__ int windows() const { return 0; }
    __device__ __forceinline__ void meta(int col0, int n, int, int* s_meta, int*) const
    {
        if ((int)threadIdx.x < n) s_meta[threadIdx.x] = col0 + (int)threadIdx.x < n_col ? cmeta[col0 + threadIdx.x] : 0;
    }
    template <class G> __device__ __forceinline__ void first(int col0, unsigned char* s_x) const
    {
        for (int p = threadIdx.x; p < G::ROWS * NKF * 4; p += PN_THREADS) {
            const int row = p / (NKF * 4), rem = p - row * (NKF * 4), cf = rem >> 2, gg = rem & 3, col = col0 + row;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (col >= 0 && col < n_col) v = X[xfrag(NKF, col >> 4, cf, (col & 15) + 16 * gg)];
            *reinterpret_cast<uint4*>(&s_x[chain_at<G>(rem, row)]) = v;
        }
    }
    static constexpr bool HALO = false;
    __device__ __forceinline__ bool goes_on(int) const { return true; }
    __device__ __forceinline__ ChainWeights weights(int rt, int wave) const
    {
        const int rt_all = rt * WG_RTS + wave % WG_RTS, rw = rt_all % (ENC_GATES / 16);
        return ChainWeights(rt_all / (ENC_GATES / 16) ? W1 : W0, NKF, rw, 0, 1);
    }
    template <class G>
    __device__ __forceinline__ void fetch(int, int rt, const int*, floatx4& bias, floatx4&) const
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), rt_all = rt * WG_RTS + wave % WG_RTS, rw = rt_all % (ENC_GATES / 16);
        bias = *reinterpret_cast<const floatx4*>((rt_all / (ENC_GATES / 16) ? b1 : b0) + rw * 16 + 4 * (threadIdx.x >> 4 & 3));
    }
    template <class G, int NA>
    __device__ __forceinline__ void last(int col0, int rt, const uint4 (&a)[NA], const floatx4& bias, const floatx4&, const unsigned char* s_x, floatx4 (*)[G::CT][64],
                                         const int (&)[G::CT], const int*) const
    {
        constexpr int CT = G::CT;
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, jl = lane & 15, g = lane >> 4;
        const int rt_all = rt * WG_RTS + wave % WG_RTS, dir = rt_all / (ENC_GATES / 16), rw = rt_all % (ENC_GATES / 16);
#pragma unroll
        for (int c0 = 0; c0 < CT; c0 += PER) {
            const int c = c0 + wave / WG_RTS, col = col0 + c * 16 + jl;
            if (c >= CT) break;
            floatx4 acc = bias;
#pragma unroll
            for (int i = 0; i < NKF; ++i)
                acc = mfma_frag<XT>(a[i], *reinterpret_cast<const uint4*>(&s_x[chain_at<G>(i * 4 + g, PN_HALO + c * 16 + jl)]), acc);
            if (col < n_col) *reinterpret_cast<floatx4*>(Y + ((size_t)dir * max_tokens + col) * ENC_GATES + rw * 16 + 4 * g) = acc;
        }
    }
};

// The recurrence with two-byte weights: one workgroup per direction and REQUEST, the direction's whole matrix (512 KB)
// resident in its CU, so a step touches no memory beyond the request's precomputed input projection.  A request's steps are a
// chain, and a chain is as fast alone on a CU as it gets; it does not depend on its companions in the call.
//
// The matrix-vector product of a step runs on the SPARSE matrix instruction: v_smfmac_f32_16x16x64_f16 contracts 64 k of a
// dense 64 x 16 operand in the 16 cycles in which the dense instruction contracts 32, its other operand holding two of every
// four k per row.  Here the dense operand is the weights (16 gate rows as its columns) and the sparse one is h: even rows
// carry k 0, 1 of every four and odd rows k 2, 3, so that the sum of two rows is the whole product - 1024 weights per
// instruction, 64 a cycle and SIMD, twice what a dense MFMA with one request in its sixteen columns, or a dot-product
// instruction of the vector units (v_dot2_f32_f16), consumes.  fp16 products, fp32 accumulation, like those.
// Four waves, one per SIMD, 64 units each.  A tile = one gate of 16 units, so the lane group q of a wave finds the four gate
// sums of its unit in the tiles 4 q .. 4 q + 3 (all four groups of a tile's rows hold the same sums: a select, no exchange)
// and updates the cell where they are.  Of a group's 16 fragments (8 registers a lane each) three are read from LDS every
// step, the others live in registers: 512 KB of registers and 160 KB of LDS are all a CU has, and LDS reads are not free (a
// fragment of every wave takes 64 cycles).  The floor of a step is 64 x 16 cycles of the matrix pipe, 0.43 us; the cell
// update, the barrier and the read of h from LDS follow it.
// Measured: one request of 165 tokens 236 us (1.41 us a step) as chains of v_dot2_f32_f16 with two threads a unit -> 117 us
// (0.67 us a step behind 6.6 us that load the weights); 16 requests of 300 tokens 206 us.  With the instructions scheduled by
// the compiler: 165 us.
// grid = (2 directions, requests), 256 threads.
constexpr int ENC_SP_THREADS = 256;
constexpr int ENC_SP_LDS_TILES = 3;                                        // of a group's sixteen fragments, those that live in LDS
constexpr int ENC_SP_W_VECS = 4 * 4 * ENC_SP_LDS_TILES * 2 * 64;           // waves x groups x fragments x 2 x lanes
constexpr int ENC_SP_LDS_BYTES = ENC_SP_W_VECS * 16 + 2 * ENC_HID * 2;
constexpr int ENC_SP_AHEAD = 2;                                            // steps between the request for an input projection and its use

// The products of one step as one run of instructions.  Left to itself the compiler moves accumulators between the two halves
// of the register file around every chain, and every move waits for the matrix pipe; here nothing does:
//   * the four chains of a group (one per gate) are interleaved, a sum is fed again after three other instructions;
//   * the groups use two sets of accumulators in turn (v[224:239], v[240:255]); a group adds up the previous group's sums and
//     clears them between its own instructions, while the vector units have nothing else to do (two of a lane's four rows
//     are enough: the other two repeat them and are never read);
//   * three of a group's sixteen fragments live in LDS; each is requested some thirteen matrix instructions (208 cycles) before
//     its use, into the registers (v[200:223]) its predecessor has just left.  In the later groups they come earlier
//     (enc_sp_piece), so that the last request of a step, for the next step's first group, is seven instructions from the
//     step's end; h arrives piece by piece.
// The hardware does not check these distances: a sum is read at least 8 wait states (gfx950: 4 passes + 4; every instruction
// in between counted as one) after the instruction that completed it, and an operand of a matrix instruction is written at
// least two wait states before.  LDS returns in order: the counts are those of the reads issued since.  Every read is waited
// for inside the run: the compiler takes its outputs as written, and may copy or spill them behind it.
#define SP_STR2(x) #x
#define SP_STR(x) SP_STR2(x)
#define SP_MM(acc, f, w) "v_smfmac_f32_16x16x64_f16 " acc ", %[h" #f "], " w ", %[ix]\n\t"
#define SP_I(U, g, f, acc) SP_MM(acc, f, "%[w" #U #f #g "]")
#define SP_WAIT(n) "s_waitcnt lgkmcnt(" #n ")\n\t"
#define SP_READ(lo, hi, next, g) "ds_read_b128 " lo ", %[la] offset:(" #next "*3+" #g ")*2048\n\tds_read_b128 " hi ", %[la] offset:(" #next "*3+" #g ")*2048+1024\n\t"
// one instruction of group U, k piece f, gate g: weights in registers (R) or the LDS-resident piece 0, 1, 2 (L0, L1, L2), whose
// successor, group N's, is requested behind it
#define SP_DO_R(U, N, f, g, acc, wait) SP_I(U, g, f, acc)
#define SP_DO_L0(U, N, f, g, acc, wait) wait SP_MM(acc, f, "v[200:207]") SP_READ("v[200:203]", "v[204:207]", N, 0)
#define SP_DO_L1(U, N, f, g, acc, wait) wait SP_MM(acc, f, "v[208:215]") SP_READ("v[208:211]", "v[212:215]", N, 1)
#define SP_DO_L2(U, N, f, g, acc, wait) wait SP_MM(acc, f, "v[216:223]") SP_READ("v[216:219]", "v[220:223]", N, 2)
#define SP_P0 "v[224:227]"
#define SP_P1 "v[228:231]"
#define SP_P2 "v[232:235]"
#define SP_P3 "v[236:239]"
#define SP_Q0 "v[240:243]"
#define SP_Q1 "v[244:247]"
#define SP_Q2 "v[248:251]"
#define SP_Q3 "v[252:255]"
#define SP_TAKE(g, r0, r1, m) "v_add_f32 %[t], v" #r0 ", v" #r1 "\n\tv_cndmask_b32 %[s" #g "], %[s" #g "], %[t], %[" m "]\n\t"
#define SP_CLEAR(r0, r1) "v_mov_b32 v" #r0 ", 0\n\tv_mov_b32 v" #r1 ", 0\n\t"
#define SP_TAKE_P0(m) SP_TAKE(0, 224, 225, m)
#define SP_TAKE_P1(m) SP_TAKE(1, 228, 229, m)
#define SP_TAKE_P2(m) SP_TAKE(2, 232, 233, m)
#define SP_TAKE_P3(m) SP_TAKE(3, 236, 237, m)
#define SP_TAKE_Q0(m) SP_TAKE(0, 240, 241, m)
#define SP_TAKE_Q1(m) SP_TAKE(1, 244, 245, m)
#define SP_TAKE_Q2(m) SP_TAKE(2, 248, 249, m)
#define SP_TAKE_Q3(m) SP_TAKE(3, 252, 253, m)
#define SP_NO_TAKE0(m)
#define SP_NO_TAKE1(m)
#define SP_NO_TAKE2(m)
#define SP_NO_TAKE3(m)
#define SP_CLEAR_P0 SP_CLEAR(224, 225)
#define SP_CLEAR_P1 SP_CLEAR(228, 229)
#define SP_CLEAR_P2 SP_CLEAR(232, 233)
#define SP_CLEAR_P3 SP_CLEAR(236, 237)
#define SP_CLEAR_Q0 SP_CLEAR(240, 241)
#define SP_CLEAR_Q1 SP_CLEAR(244, 245)
#define SP_CLEAR_Q2 SP_CLEAR(248, 249)
#define SP_CLEAR_Q3 SP_CLEAR(252, 253)
// U: group, N: the group behind it, C: its accumulators (P or Q), O: the previous group's, TAKE, m: how the previous group's
// sums are taken; W0 .. W3: waits for the pieces of h, WL: wait for an LDS-resident piece; Xfg: where the weights of k piece f,
// gate g are
#define SP_GROUP(U, N, C, O, TAKE, m, W0, W1, W2, W3, WL, X00, X01, X02, X03, X10, X11, X12, X13, X20, X21, X22, X23, X30, X31, X32, X33) \
    W0 SP_DO_##X00(U, N, 0, 0, SP_##C##0, WL) SP_DO_##X01(U, N, 0, 1, SP_##C##1, WL) SP_DO_##X02(U, N, 0, 2, SP_##C##2, WL)              \
    SP_DO_##X03(U, N, 0, 3, SP_##C##3, WL)                                                                                               \
    W1 SP_DO_##X10(U, N, 1, 0, SP_##C##0, WL) TAKE##0(m) SP_DO_##X11(U, N, 1, 1, SP_##C##1, WL) TAKE##1(m)                               \
    SP_DO_##X12(U, N, 1, 2, SP_##C##2, WL) TAKE##2(m) SP_DO_##X13(U, N, 1, 3, SP_##C##3, WL) TAKE##3(m)                                  \
    W2 SP_DO_##X20(U, N, 2, 0, SP_##C##0, WL) SP_CLEAR_##O##0 SP_DO_##X21(U, N, 2, 1, SP_##C##1, WL) SP_CLEAR_##O##1                     \
    SP_DO_##X22(U, N, 2, 2, SP_##C##2, WL) SP_CLEAR_##O##2 SP_DO_##X23(U, N, 2, 3, SP_##C##3, WL) SP_CLEAR_##O##3                        \
    W3 SP_DO_##X30(U, N, 3, 0, SP_##C##0, WL) SP_DO_##X31(U, N, 3, 1, SP_##C##1, WL) SP_DO_##X32(U, N, 3, 2, SP_##C##2, WL)              \
    SP_DO_##X33(U, N, 3, 3, SP_##C##3, WL)
#define SP_STEP(hoff)                                                                                                                    \
    SP_WAIT(0)                                                                                                                           \
    "ds_read_b128 %[h0], %[ha] offset:" SP_STR(hoff) "\n\tds_read_b128 %[h1], %[ha] offset:" SP_STR(hoff) "+128\n\t"                    \
    "ds_read_b128 %[h2], %[ha] offset:" SP_STR(hoff) "+256\n\tds_read_b128 %[h3], %[ha] offset:" SP_STR(hoff) "+384\n\t"                \
    SP_GROUP(0, 1, P, Q, SP_NO_TAKE, "", SP_WAIT(3), SP_WAIT(2), SP_WAIT(3), SP_WAIT(4), , R, R, R, R, L0, R, R, R, R, L1, R, R, R, R, L2, R) \
    SP_GROUP(1, 2, Q, P, SP_TAKE_P, "m0", , , , , SP_WAIT(4), R, R, R, R, L0, R, R, R, R, L1, R, R, R, R, L2, R)                          \
    SP_GROUP(2, 3, P, Q, SP_TAKE_Q, "m1", , , , , SP_WAIT(4), R, R, L0, R, R, R, R, L1, R, R, R, L2, R, R, R, R)                          \
    SP_GROUP(3, 0, Q, P, SP_TAKE_P, "m2", , , , , SP_WAIT(4), L0, R, R, R, L1, R, R, R, L2, R, R, R, R, R, R, R)                          \
    "s_nop 4\n\t" SP_TAKE_Q0("m3") SP_TAKE_Q1("m3") SP_TAKE_Q2("m3") SP_TAKE_Q3("m3") SP_WAIT(0)
// the LDS-resident pieces, as the groups above have them: the number of k piece f of gate g in group U, or -1
__device__ constexpr int enc_sp_piece(int U, int f, int g)
{
    constexpr int at[4][ENC_SP_LDS_TILES] = {{4, 9, 14}, {4, 9, 14}, {2, 7, 11}, {0, 4, 8}};      // 4 f + g
    for (int i = 0; i < ENC_SP_LDS_TILES; ++i)
        if (at[U][i] == 4 * f + g) return i;
    return -1;
}
// register operands: %[wUfg] = k piece f of gate g in group U; the first 32 fragments in the accumulation half of the file
#define SP_W(c, U, f, g) [w##U##f##g] c(wr[U][f][g])
#define SP_WGROUP01(U)                                                                                                                   \
    SP_W("a", U, 0, 0), SP_W("a", U, 0, 1), SP_W("a", U, 0, 2), SP_W("a", U, 0, 3), SP_W("a", U, 1, 1), SP_W("a", U, 1, 2),               \
        SP_W("a", U, 1, 3), SP_W("a", U, 2, 0), SP_W("a", U, 2, 2), SP_W("a", U, 2, 3), SP_W("a", U, 3, 0), SP_W("a", U, 3, 1),           \
        SP_W("a", U, 3, 3)
#define SP_WGROUP2                                                                                                                       \
    SP_W("a", 2, 0, 0), SP_W("a", 2, 0, 1), SP_W("a", 2, 0, 3), SP_W("a", 2, 1, 0), SP_W("a", 2, 1, 1), SP_W("a", 2, 1, 2),               \
        SP_W("v", 2, 2, 0), SP_W("v", 2, 2, 1), SP_W("v", 2, 2, 2), SP_W("v", 2, 3, 0), SP_W("v", 2, 3, 1), SP_W("v", 2, 3, 2),           \
        SP_W("v", 2, 3, 3)
#define SP_WGROUP3                                                                                                                       \
    SP_W("v", 3, 0, 1), SP_W("v", 3, 0, 2), SP_W("v", 3, 0, 3), SP_W("v", 3, 1, 1), SP_W("v", 3, 1, 2), SP_W("v", 3, 1, 3),               \
        SP_W("v", 3, 2, 1), SP_W("v", 3, 2, 2), SP_W("v", 3, 2, 3), SP_W("v", 3, 3, 0), SP_W("v", 3, 3, 1), SP_W("v", 3, 3, 2),           \
        SP_W("v", 3, 3, 3)
#define SP_RUN(hoff)                                                                                                                     \
    asm volatile(SP_STEP(hoff)                                                                                                           \
                 : [h0] "=&v"(hv[0]), [h1] "=&v"(hv[1]), [h2] "=&v"(hv[2]), [h3] "=&v"(hv[3]), [s0] "+v"(gs[0]), [s1] "+v"(gs[1]),         \
                   [s2] "+v"(gs[2]), [s3] "+v"(gs[3]), [t] "=&v"(tmp), "+{v[200:207]}"(wv[0]), "+{v[208:215]}"(wv[1]),                    \
                   "+{v[216:223]}"(wv[2]), "+{v[224:227]}"(accp[0]), "+{v[228:231]}"(accp[1]), "+{v[232:235]}"(accp[2]),                  \
                   "+{v[236:239]}"(accp[3]), "+{v[240:243]}"(accq[0]), "+{v[244:247]}"(accq[1]), "+{v[248:251]}"(accq[2]),                \
                   "+{v[252:255]}"(accq[3])                                                                                               \
                 : [ha] "v"(h_at), [la] "v"(w_at), [ix] "v"(idx), [m0] "s"(lanes_of(0)), [m1] "s"(lanes_of(1)), [m2] "s"(lanes_of(2)),     \
                   [m3] "s"(lanes_of(3)), SP_WGROUP01(0), SP_WGROUP01(1), SP_WGROUP2, SP_WGROUP3                                          \
                 : "memory")

typedef uint32_t u32x8_t __attribute__((ext_vector_type(8)));

__global__ __launch_bounds__(ENC_SP_THREADS) void k_enc_lstm_sp(const uint4* __restrict__ Whh0, const uint4* __restrict__ Whh1,
                                                                const float* __restrict__ xproj, PnWindows w, int max_tokens, float* __restrict__ out)
{
    constexpr int NK = ENC_HID / 32, NF = ENC_HID / 64;                    // dense fragments of the stored matrix, k pieces of 64
    static_assert(NF == 4, "the instruction runs are written for four pieces of k");
    extern __shared__ uint4 lds_enc[];
    uint4* wl = lds_enc;
    uint16_t* hs = reinterpret_cast<uint16_t*>(lds_enc + ENC_SP_W_VECS);   // h as halves, [buffer][unit in operand order]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 15, q = lane >> 4;
    const int dir = blockIdx.x, req = blockIdx.y;
    const int len = __builtin_amdgcn_readfirstlane((int)w.len[req]), col0 = __builtin_amdgcn_readfirstlane(w.col0[req]);
    const uint4* Wl = (dir ? Whh1 : Whh0) + lane;
    uint4* wlw = wl + wave * 4 * ENC_SP_LDS_TILES * 2 * 64 + lane;
    // tile 4 (4 wave + U) + g = gate g of the units 16 (4 wave + U) ..; its k piece f = the dense fragments 2 f and 2 f + 1
    u32x8_t wr[4][NF][4];
#pragma unroll
    for (int U = 0; U < 4; ++U)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const size_t at = ((size_t)(4 * (4 * wave + U) + g) * NK + 2 * f) * 64;
                const uint4 lo = Wl[at], hi = Wl[at + 64];
                const int piece = enc_sp_piece(U, f, g);
                if (piece >= 0) {                                  // (lives in LDS)
                    wlw[((U * ENC_SP_LDS_TILES + piece) * 2) * 64] = lo;
                    wlw[((U * ENC_SP_LDS_TILES + piece) * 2 + 1) * 64] = hi;
                } else {
                    wr[U][f][g] = u32x8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                }
            }
    reinterpret_cast<uint32_t*>(hs)[tid] = 0;                              // h = 0, both buffers

    // this lane's unit, and where its h lies in the sparse operand: k = 64 f + 16 q' + 4 j + 2 p + e sits in piece (f, q', p),
    // half 2 j + e; a lane of row r reads the pieces of parity p = r % 2
    const int unit = 16 * (4 * wave + q) + n;
    const int hpos = ((unit >> 4) * 2 + ((n >> 1) & 1)) * 8 + 2 * (n >> 2) + (n & 1);
    const int idx = (n & 1) ? (int)0xEEEEEEEEu : 0x44444444;
    // Input projections and F_enc through bounds-checked descriptors: steps past the request's end (the loop below takes
    // ENC_SP_AHEAD at a time) read zeros and store nothing.
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(xproj) + ((size_t)dir * max_tokens + col0) * ENC_GATES, 0,
                                                                        len * ENC_GATES * 4, BUFFER_RSRC_RAW);
    const __amdgpu_buffer_rsrc_t outr = __builtin_amdgcn_make_buffer_rsrc(out + (size_t)col0 * (2 * ENC_HID), 0, len * 2 * ENC_HID * 4, BUFFER_RSRC_RAW);
    const int step = dir ? -1 : 1;
    int tok = dir ? len - 1 : 0;                                           // of the next step; leaves 0 .. len - 1 at the request's end
    auto load_x = [&](int t) { return __builtin_bit_cast(floatx4, buffer_load16(xr, (t * ENC_GATES + 4 * unit) * 4)); };
    floatx4 x[ENC_SP_AHEAD];
#pragma unroll
    for (int j = 0; j < ENC_SP_AHEAD; ++j) x[j] = load_x(tok + j * step);
    float c = 0.f;
    floatx4 accp[4], accq[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) accp[g] = accq[g] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto lanes_of = [](int group) { return 0xFFFFull << (16 * group); };
    typedef __attribute__((address_space(3))) void lds_void;
    const uint32_t w_at = (uint32_t)(uintptr_t)(lds_void*)wlw, h_at = (uint32_t)(uintptr_t)(lds_void*)(hs + (q * 2 + (n & 1)) * 8);
    u32x8_t wv[ENC_SP_LDS_TILES];
#pragma unroll
    for (int g = 0; g < ENC_SP_LDS_TILES; ++g) {
        const uint4 lo = wlw[g * 2 * 64], hi = wlw[(g * 2 + 1) * 64];      // (this wave's own writes)
        wv[g] = u32x8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    }
    // every weight has arrived before the loop, and so have the first projections: the loop's waits count its own requests only
#pragma unroll
    for (int U = 0; U < 4; ++U)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                if (enc_sp_piece(U, f, g) < 0) {
                    if (U < 2 || (U == 2 && f < 2)) asm volatile("" : "+a"(wr[U][f][g]));
                    else asm volatile("" : "+v"(wr[U][f][g]));
                }
    vm_in_flight_at_most<0>();
    __syncthreads();

    for (int s0 = 0; s0 < len; s0 += ENC_SP_AHEAD) {
#pragma unroll
        for (int j = 0; j < ENC_SP_AHEAD; ++j) {
            u32x4_t hv[NF];
            floatx4 gs = {0.f, 0.f, 0.f, 0.f};
            float tmp;
            if (j & 1) SP_RUN(512);
            else SP_RUN(0);
            gs += x[j];
            const float gi = sigmoidf_(gs[0]), gf = sigmoidf_(gs[1]), gg = tanhf_(gs[2]), go = sigmoidf_(gs[3]);
            c = gf * c + gi * gg;
            const float h = go * tanhf_(c);
            hs[((j + 1) & 1) * ENC_HID + hpos] = from_float<h16_t>(h).bits;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(h), outr, (tok * 2 * ENC_HID + dir * ENC_HID + unit) * 4, 0, 0);
            x[j] = load_x(tok + ENC_SP_AHEAD * step);
            tok += step;
            __syncthreads();                              // h is complete (the other buffer is free for the next step)
        }
    }
}
#undef SP_STR
#undef SP_MM
#undef SP_I
#undef SP_WAIT
#undef SP_READ
#undef SP_TAKE
#undef SP_CLEAR
#undef SP_GROUP
#undef SP_STEP
#undef SP_RUN
#undef SP_W

// The recurrence with fp32 weights: a direction's matrix (1 MB) does not fit a CU, and streaming it from L2 takes 29 us a step
// (k_enc_lstm_alone; one CU's load path).  So G workgroups share a direction of R requests: each keeps the gate rows of 256 / G
// units in registers (64 a thread), forms those units' gate sums from the whole h, updates their cells, and hands their h to its
// partners through memory.  h needs no separate flag: |h| <= 1 leaves bit 30 of its fp32 word free, which carries the round
// of the word's reuse (two buffers per request, the bit flips each time a buffer comes round; k_enc_embed clears the words
// of a call).  A partner can be at most one step behind: nobody finishes step s + 1 without all of its words of step s.
// A step is bound by that exchange (a store becoming visible plus a trip of the poll, about 1 us); the products take 0.1 us
// (16 threads per unit, each 16 k of its four gate rows: 64 FMAs) to 0.4 us (16 waves a workgroup).  Measured: one request of
// 165 tokens 0.24 ms (1.4 us a step; 6.6 ms with the matrix streamed through MFMAs whose columns were the requests), 8 requests
// of 30 .. 300 tokens 0.41 ms, 60 of them 0.94 ms (two to a group of workgroups).  G is as large as the number of workgroups
// allows: all of them (2 directions x groups x G <= one per CU) must be resident at once, because they
// wait for each other.  Work on other streams may keep some from starting (a second encoder, a pool whose own workgroups
// wait for each other): every wait is bounded, one that runs out raises *fault and ends the workgroup, and k_enc_lstm_alone
// behind this kernel then forms the call's results without waiting for anybody.
// A unit's sum is taken in the same order whatever G and R are, so a request's result does not depend on its companions.
// grid = (G, groups of R requests, 2 directions), 4096 / G threads (<= 1024).
constexpr int ENC_X_PARTS = 16;                                            // threads per unit: thread p owns k = 64 i + 4 p .. + 3
constexpr uint32_t ENC_X_ROUND = 1u << 30;

template <int CTRL> __device__ __forceinline__ float dpp_add(float x)
{
    return x + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, true));
}
// The four gate sums of a unit over this lane's 16 k; weights(g, i) = four k of gate g.  One order of the sums and one form of
// the cell for both kernels, so that they agree bit for bit.
constexpr int ENC_X_NI = ENC_HID / (4 * ENC_X_PARTS);
template <typename W>
__device__ __forceinline__ floatx4 gate_parts(const float* h, int p, W&& weights)
{
    const float4* h4 = reinterpret_cast<const float4*>(h);
    floatx4 gs = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < ENC_X_NI; ++i) {
        const float4 hv = h4[i * ENC_X_PARTS + p];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 w = weights(g, i);
            gs[g] = fmaf(w.w, hv.w, fmaf(w.z, hv.z, fmaf(w.y, hv.y, fmaf(w.x, hv.x, gs[g]))));
        }
    }
    return gs;
}
__device__ __forceinline__ float cell(floatx4 gs, float& c)
{
    const float gi = sigmoidf_(gs[0]), gf = sigmoidf_(gs[1]), gg = tanhf_(gs[2]), go = sigmoidf_(gs[3]);
    c = fmaf(gf, c, gi * gg);
    return go * tanhf_(c);
}

// the sum over the 16 lanes of a row, the same bits in all of them (partners add the same two values at every level)
__device__ __forceinline__ float row16_sum(float x)
{
    x = dpp_add<0xB1>(x);          // quad_perm 1 0 3 2
    x = dpp_add<0x4E>(x);          // quad_perm 2 3 0 1
    x = dpp_add<0x141>(x);         // row_half_mirror
    return dpp_add<0x140>(x);      // row_mirror
}

template <int R>
__global__ __launch_bounds__(1024) void k_enc_lstm_shared(const uint4* __restrict__ Whh0, const uint4* __restrict__ Whh1,
                                                          const float* __restrict__ xproj, uint32_t* hx, PnWindows w, int max_tokens,
                                                          float* __restrict__ out, int wait_polls, int* fault)
{
    constexpr int NK = ENC_HID / 16, NI = ENC_X_NI;
    __shared__ __attribute__((aligned(16))) float hs[2][R][ENC_HID];
    __shared__ int gave_up[2];                         // by the parity of the step: what a wave reads behind a step's barrier is not
                                                       // written again before that wave has passed the next one
    const int tid = threadIdx.x, nthr = blockDim.x, p = tid & (ENC_X_PARTS - 1);
    const int dir = blockIdx.z, req0 = blockIdx.y * R, unit = blockIdx.x * (nthr / ENC_X_PARTS) + tid / ENC_X_PARTS;
    // lengths and first tokens once, into registers: the request table is a kernel argument
    int len[R], col0[R], lmax = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int rq = min(req0 + r, w.n - 1);
        len[r] = req0 + r < w.n ? (int)w.len[rq] : 0;
        col0[r] = w.col0[rq];
        lmax = max(lmax, len[r]);
    }
    const uint4* Whh = dir ? Whh1 : Whh0;
    float4 wr[4][NI];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int i = 0; i < NI; ++i)
            wr[g][i] = __builtin_bit_cast(float4, Whh[xfrag(NK, unit >> 2, 4 * i + (p >> 2), 4 * (unit & 3) + g + 16 * (p & 3))]);
    for (int i = tid; i < 2 * R * ENC_HID; i += nthr) (&hs[0][0][0])[i] = 0.f;
    if (tid < 2) gave_up[tid] = 0;

    auto token = [&](int r, int s) { return min(max(dir ? len[r] - 1 - s : s, 0), max(len[r] - 1, 0)); };
    const float* xp = xproj + (size_t)dir * max_tokens * ENC_GATES + 4 * unit;
    uint32_t* words = hx + ((size_t)dir * w.n + req0) * 2 * ENC_HID;       // [request][buffer][unit]
    floatx4 x[R];
    float c[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        x[r] = *reinterpret_cast<const floatx4*>(xp + (size_t)(col0[r] + token(r, 0)) * ENC_GATES);
        c[r] = 0.f;
    }
    __syncthreads();

    for (int s = 0; s < lmax; ++s) {
        const int buf = s & 1;
        const uint32_t round = ((s >> 1) & 1) ? 0u : ENC_X_ROUND;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (s >= len[r]) continue;                                     // uniform over the workgroup and its partners
            floatx4 gs = gate_parts(&hs[buf][r][0], p, [&](int g, int i) { return wr[g][i]; });
#pragma unroll
            for (int g = 0; g < 4; ++g) gs[g] = row16_sum(gs[g]);
            gs += x[r];
            const float h = cell(gs, c[r]);
            if (p == 0) {
                if (s + 1 < len[r])
                    __hip_atomic_store(&words[(r * 2 + buf) * ENC_HID + unit], (__float_as_uint(h) & ~ENC_X_ROUND) | round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                out[(size_t)(col0[r] + token(r, s)) * (2 * ENC_HID) + dir * ENC_HID + unit] = h;
            }
            x[r] = *reinterpret_cast<const floatx4*>(xp + (size_t)(col0[r] + token(r, s + 1)) * ENC_GATES);
        }
        // the whole h of this step, for the next one
        for (int i = tid; i < R * ENC_HID; i += nthr) {
            const int r = i / ENC_HID, u = i - r * ENC_HID;
            int l = len[0];
#pragma unroll
            for (int k = 1; k < R; ++k) l = r == k ? len[k] : l;
            if (s + 1 >= l) continue;
            uint32_t* at = &words[(r * 2 + buf) * ENC_HID + u];
            uint32_t v = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int polls = 0; (v & ENC_X_ROUND) != round; ++polls) {
                if (polls >= wait_polls) {
                    gave_up[buf] = 1;
                    __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                v = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            v &= ~ENC_X_ROUND;
            if ((v & 0x7FFFFFFFu) >= 0x3FC00000u) v |= ENC_X_ROUND;        // no h has a magnitude of 1.5: it was a NaN
            hs[buf ^ 1][r][u] = __uint_as_float(v);
        }
        __syncthreads();                               // h is complete (every wave has read the other buffer)
        if (gave_up[buf]) return;                      // every wave of the workgroup, at the same step
    }
}

// The same recurrence by one workgroup per direction and request, the weights streamed from L2 in every step (28.7 us a step: one
// CU's load path; 60 requests of 30 .. 300 tokens side by side 8.5 ms).  It ends at once unless k_enc_lstm_shared gave up (given
// == nullptr: it was not launched, the device has too few compute units for its workgroups).
// grid = (2 directions, requests), 1024 threads.
__global__ __launch_bounds__(1024) void k_enc_lstm_alone(const uint4* __restrict__ Whh0, const uint4* __restrict__ Whh1,
                                                         const float* __restrict__ xproj, PnWindows w, int max_tokens,
                                                         float* __restrict__ out, const int* given)
{
    constexpr int NK = ENC_HID / 16, PASS = 1024 / ENC_X_PARTS, NP = ENC_HID / PASS;
    if (given && *given == 0) return;
    __shared__ __attribute__((aligned(16))) float hs[2][ENC_HID], cs[ENC_HID];
    const int tid = threadIdx.x, p = tid & (ENC_X_PARTS - 1), dir = blockIdx.x;
    const int len = (int)w.len[blockIdx.y], col0 = w.col0[blockIdx.y];
    const uint4* Whh = dir ? Whh1 : Whh0;
    if (tid < ENC_HID) hs[0][tid] = cs[tid] = 0.f;
    __syncthreads();
    for (int s = 0; s < len; ++s) {
        const size_t col = (size_t)col0 + (dir ? len - 1 - s : s);
#pragma unroll 1
        for (int k = 0; k < NP; ++k) {                 // (a pass's weights are all the registers hold)
            const int unit = k * PASS + tid / ENC_X_PARTS;
            floatx4 gs = gate_parts(hs[s & 1], p, [&](int g, int i) {
                return __builtin_bit_cast(float4, Whh[xfrag(NK, unit >> 2, 4 * i + (p >> 2), 4 * (unit & 3) + g + 16 * (p & 3))]);
            });
#pragma unroll
            for (int g = 0; g < 4; ++g) gs[g] = row16_sum(gs[g]);
            gs += *reinterpret_cast<const floatx4*>(xproj + ((size_t)dir * max_tokens + col) * ENC_GATES + 4 * unit);
            float c = cs[unit];                        // (read and written by the lanes of one wave)
            const float h = cell(gs, c);
            if (p == 0) {
                cs[unit] = c;
                hs[(s + 1) & 1][unit] = h;
                out[col * (2 * ENC_HID) + dir * ENC_HID + unit] = h;
            }
        }
        __syncthreads();                               // h is complete (every wave has read the other buffer)
    }
}

template <int R>
void lstm_shared(int G, const EncoderPtrs& d, const PnWindows& w, float* out, hipStream_t s)
{
    hipLaunchKernelGGL((k_enc_lstm_shared<R>), dim3(G, (w.n + R - 1) / R, 2), dim3(ENC_HID / G * ENC_X_PARTS), 0, s, (const uint4*)d.w_hh[0],
                       (const uint4*)d.w_hh[1], d.xproj, d.hx, w, d.max_tokens, out, d.wait_polls, d.gave_up);
}

template <typename XT>
hipError_t front_by_layers(const EncoderPtrs& d, int n_col, hipStream_t s)
{
    constexpr int C = ENC_DIM;
    static_assert(enc_chain_columns(sizeof(XT)) / 16 + 1 >= cols_from<XT, C, C, PN_TAPS>(), "calls with layers of their own take k_conv_cols");
    const int n_ctiles = (n_col + 15) / 16;
    ColArgs p{};
    p.cmeta = d.cmeta;
    p.n_ctiles = n_ctiles;
    hipError_t e = hipSuccess;
    for (int l = 0; l < ENC_CONVS && e == hipSuccess; ++l) {
        p.W = (const uint4*)d.conv_w[l];
        p.bias = d.conv_b[l];
        p.Xin = (const uint4*)d.act[l & 1];
        p.Xout = d.act[(l & 1) ^ 1];
        e = conv_cols<XT, C, C, PN_TAPS, CC_RELU>(p, s);
    }
    if (e != hipSuccess) return e;
    const void* x1 = d.act[1];
    if constexpr (enc_chain_columns(sizeof(XT)) / 16 + 1 < cols_from<XT, C, 2 * ENC_GATES, 1>())
        if (n_ctiles < cols_from<XT, C, 2 * ENC_GATES, 1>()) {
            hipLaunchKernelGGL((k_enc_xproj<XT>), dim3(ENC_GATES / 16 / 4, n_ctiles, 2), dim3(256), 0, s, (const uint4*)d.w_ih[0], (const uint4*)d.w_ih[1],
                               d.b[0], d.b[1], (const uint4*)x1, n_col, d.max_tokens, d.xproj);
            return hipGetLastError();
        }
    p.W = (const uint4*)d.w_ih[0];
    p.W1 = (const uint4*)d.w_ih[1];
    p.bias = d.b[0];
    p.bias1 = d.b[1];
    p.Xin = (const uint4*)x1;
    p.Xout = nullptr;
    p.out = d.xproj;
    p.n_col = n_col;
    p.max_cols = d.max_tokens;
    return conv_cols<XT, C, 2 * ENC_GATES, 1, CC_XPROJ>(p, s);
}

template <typename XT>
hipError_t front_as_one(const EncoderPtrs& d, int n_col, hipStream_t s)
{
    EncChain<XT> job;
    job.X = (const uint4*)d.act[0];
    job.cmeta = d.cmeta;
    job.n_col = n_col;
    job.max_tokens = d.max_tokens;
    job.W0 = (const uint4*)d.w_ih[0];
    job.W1 = (const uint4*)d.w_ih[1];
    job.b0 = d.b[0];
    job.b1 = d.b[1];
    job.Y = d.xproj;
    ChainArgs p{};
    for (int l = 0; l < ENC_CONVS; ++l) {
        p.W[l] = (const uint4*)d.conv_w[l];
        p.b[l] = d.conv_b[l];
    }
    p.words = d.chain_words;
    p.set_bytes = d.chain_set_bytes;
    p.state = d.chain_state;
    p.polls = d.wait_polls < CHAIN_POLLS ? d.wait_polls : CHAIN_POLLS;
    return conv_chain<XT, enc_chain_columns(sizeof(XT))>(job, p, n_col, s);
}

template <typename XT>
hipError_t run_typed(const EncoderPtrs& d, const PnWindows& w, int n_col, const EncStaged& staged, float* out, hipStream_t s)
{
    const int n_ctiles = (n_col + 15) / 16, n_col_pad = n_ctiles * 16;
    XT* x0 = reinterpret_cast<XT*>(d.act[0]);
    EncTables tb;
    for (int t = 0; t < ENC_TABLES; ++t) tb.t[t] = d.tables[t];
    hipLaunchKernelGGL((k_enc_embed<XT>), dim3((n_col_pad + 3) / 4), dim3(256), 0, s, tb, staged, n_col, n_col_pad, x0, d.cmeta, d.hx,
                       sizeof(XT) == 2 ? 0 : w.n * 4 * ENC_HID, d.gave_up);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = n_col <= enc_chain_columns(sizeof(XT)) ? front_as_one<XT>(d, n_col, s) : front_by_layers<XT>(d, n_col, s);
    if (e != hipSuccess) return e;
    if constexpr (sizeof(XT) == 2) {
        static bool attr_set = false;               // dynamic LDS above 64 KB has to be allowed once
        if (!attr_set) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_enc_lstm_sp), hipFuncAttributeMaxDynamicSharedMemorySize, ENC_SP_LDS_BYTES);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        hipLaunchKernelGGL(k_enc_lstm_sp, dim3(2, w.n), dim3(ENC_SP_THREADS), ENC_SP_LDS_BYTES, s, (const uint4*)d.w_hh[0], (const uint4*)d.w_hh[1], d.xproj, w,
                           d.max_tokens, out);
    } else {
        // as many workgroups per direction and request as can all be resident, at least 4 (256 KB of weights each); from
        // there on, several requests per group of workgroups
        int G = 16, R = 1;
        auto wgs = [&] { return 2L * G * ((w.n + R - 1) / R); };
        while (G > 4 && wgs() > d.n_cu) G /= 2;
        while (R < 8 && wgs() > d.n_cu) R *= 2;
        const bool share = wgs() <= d.n_cu;
        if (!share) {
            // too few compute units for that many requests: without partners
        } else if (R == 1) lstm_shared<1>(G, d, w, out, s);
        else if (R == 2) lstm_shared<2>(G, d, w, out, s);
        else if (R == 4) lstm_shared<4>(G, d, w, out, s);
        else lstm_shared<8>(G, d, w, out, s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_enc_lstm_alone, dim3(2, w.n), dim3(1024), 0, s, (const uint4*)d.w_hh[0], (const uint4*)d.w_hh[1], d.xproj, w,
                           d.max_tokens, out, share ? d.gave_up : nullptr);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_encoder(const EncoderPtrs& d, int wdtype, const PnWindows& w, int n_col, const EncStaged& staged, float* out, hipStream_t s)
{
    if (n_col < 1 || w.n < 1) return hipSuccess;
    return wdtype == 0 ? run_typed<float>(d, w, n_col, staged, out, s) : run_typed<h16_t>(d, w, n_col, staged, out, s);
}

}  // namespace tts
