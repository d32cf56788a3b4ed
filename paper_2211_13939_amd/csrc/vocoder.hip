// Vocoder kernels (Sec. 2.1.4, Eq. 3, Eq. 4): the generator G as a chain of one-dimensional convolutions on
// MFMA, the splice of [tail(M_pre), M_cur] and the equal-power fade of the overlapping audio.
//
// Every convolution of G -- plain, dilated or transposed -- is one GEMM  Y[row][p] = sum_k W[row][k] X[k][p]
// over the positions p of a window, with k = tap * C_in + channel and X[k][p] = act(x[p + (tap - half) * dil][channel]):
//   plain / dilated   rows = output channels, taps = the kernel's taps
//   transposed        stride u, kernel 2u, padding u/2: output u p + r depends on inputs p - 1, p, p + 1 only, so it is
//                     a 3-tap convolution with rows = (phase r, output channel) and one zero tap per phase
// Activations live in HBM as fp32 [position][channel]; a workgroup stages the positions of its tile plus the halo
// in LDS (leaky ReLU and the conversion to the MFMA operand type happen there, once per element), so that a lane's
// B operand -- consecutive channels of one tap at one position -- is one 16-byte LDS read.  LDS holds a plane per 16
// bytes of channels.  The weights are stored in A-fragment order and stream from L2.
// Windows of different requests lie at a fixed stride; positions outside a window's own length read as zero, which
// is the zero padding of every layer.
#include <algorithm>

#include "vocoder_kernels.h"

#include "mfma.h"

namespace tts {
namespace {

constexpr int VC_THREADS = 256;
constexpr int VC_WAVES = VC_THREADS / 64;
constexpr float VC_SLOPE = 0.1f;
constexpr int VC_LDS_BYTES = 48 * 1024;
constexpr int VC_AHEAD = 4;                  // k steps between the request for a weight fragment and its use

enum { EPI_PLAIN = 0, EPI_UP = 2, EPI_POST = 3 };

template <typename XT, int CIN> struct VcGeom {
    static constexpr int EPL = Frag<XT>::EPL;
    static constexpr int GP = CIN / EPL;         // 16-byte pieces per position
    static_assert(CIN % EPL == 0, "channels must fill whole 16-byte pieces");
};

// positions per workgroup: as many as the accumulators (64 registers) and 48 KB of LDS allow
template <typename XT, int CIN, int ROWS, int HALO, bool SHORT = false> constexpr int vc_tp()
{
    constexpr int RT = ROWS / 16, RG = RT < 4 ? RT : 4;
    int tp = SHORT ? 64 : 1024 / RG;
    while (tp > 64 && (tp + 2 * HALO) * VcGeom<XT, CIN>::GP * 16 > VC_LDS_BYTES) tp /= 2;
    return tp;
}
// rows of the operand buffer: a plane per 16 bytes of channels, a multiple of 16 rows apart (see VrGeom::STRIDE)
constexpr int vc_stride(int rows) { return (rows + 15) / 16 * 16; }

struct VcArgs {
    const float* in0;     // input activations [position][C_in]
    const float* in1;     // with SRC3 the input is the mean of in0, in1, in2 (the three residual blocks of a stage)
    const float* in2;
    float* out;
    const uint4* W;
    const float* bias;
};

// slope < 1: the larger of x and slope * x.  (fmaxf costs a third instruction that quiets x first; maximum has NaN for NaN too.)
__device__ __forceinline__ float lrelu(float x) { return __builtin_elementwise_maximum(x, VC_SLOPE * x); }

template <typename XT> __device__ __forceinline__ void lds_put4(uint4* lds, int elem, float4 v);
template <> __device__ __forceinline__ void lds_put4<float>(uint4* lds, int elem, float4 v)
{
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(lds) + elem) = v;
}
template <> __device__ __forceinline__ void lds_put4<h16_t>(uint4* lds, int elem, float4 v)
{
    uint2 u;
    u.x = pack2<h16_t>(v.x, v.y);
    u.y = pack2<h16_t>(v.z, v.w);
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(lds) + elem) = u;
}

// Four channels of one position of the input: of one array, or of three whose mean is meant.
struct Quad1 {
    float4 v;
    __device__ __forceinline__ float4 value() const { return v; }
};
struct Quad3 {
    float4 v0, v1, v2;
    __device__ __forceinline__ float4 value() const
    {
        constexpr float third = 1.0f / 3.0f;
        return make_float4(((v0.x + v1.x) + v2.x) * third, ((v0.y + v1.y) + v2.y) * third, ((v0.z + v1.z) + v2.z) * third, ((v0.w + v1.w) + v2.w) * third);
    }
};

// One tile of TP positions of one window, all ROWS output rows.
//   valid  positions of this window that exist (input side); wbase = first position of the window in the arrays
//   p0     first position of the tile inside the window
//   fetch  (position that exists, channel / 4) -> Quad1 or Quad3
//   seen   (position, channel / 4, the four values): every piece that is staged, among them such as lie outside the window (values of no meaning)
//   emit   (position, sample): EPI_POST, instead of a store
template <typename XT, int CIN, int ROWS, int COUT, int KS, int TP, int EPI, bool PRE_ACT, int U, int RG, typename FETCH, typename SEEN, typename EMIT>
__device__ __forceinline__ void conv_tile(const VcArgs& a, int valid, size_t wbase, int p0, uint4* lds, FETCH fetch, SEEN seen, EMIT emit)
{
    using G = VcGeom<XT, CIN>;
    constexpr int KB = Frag<XT>::KB;
    constexpr int RT = ROWS / 16, CT = TP / (16 * VC_WAVES);
    constexpr int NK = (KS * CIN + KB - 1) / KB;     // K fragments (the weights are zero padded to whole fragments)
    constexpr int NQ = KS * G::GP;                   // 16-byte pieces of k that exist
    constexpr int C4 = CIN / 4;
    static_assert(ROWS % 16 == 0 && RT % RG == 0 && TP % (16 * VC_WAVES) == 0, "tile shape");
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    constexpr int halo = (KS - 1) / 2, nrows = TP + 2 * halo, STRIDE = vc_stride(nrows);

    // The workgroup's share of the output rows: row group blockIdx.z.  Its weights stream from L2 / HBM through a ring of registers, requested
    // VC_AHEAD k steps before they are used, or, where it has one row tile, all of them here: a window's few dozen positions leave nothing else to
    // wait behind.
    const int rt0 = blockIdx.z * RG;
    const uint4* Wl = a.W + (size_t)rt0 * NK * 64 + lane;
    constexpr int AHEAD = RG == 1 || NK < VC_AHEAD ? NK : VC_AHEAD;
    uint4 ring[AHEAD][RG];
#pragma unroll
    for (int d = 0; d < AHEAD; ++d)
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) ring[d][rg] = Wl[((size_t)rg * NK + d) * 64];

    // ---- stage positions [p0 - halo, p0 + TP + halo): activation and operand type applied once per element; a few pieces of every
    // thread are requested together, from clamped positions
    using Quad = decltype(fetch(0, 0));
    constexpr int N_STAGE = nrows * C4, AT_ONCE = sizeof(Quad) > 16 ? 4 : 8;
    for (int i0 = 0; i0 < N_STAGE; i0 += AT_ONCE * VC_THREADS) {
        Quad v[AT_ONCE];
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {
            const int idx = min(i0 + i * VC_THREADS + tid, N_STAGE - 1), row = idx / C4;
            v[i] = fetch(min(max(p0 - halo + row, 0), valid - 1), idx - row * C4);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i) {
            const int idx = i0 + i * VC_THREADS + tid, row = idx / C4, c4 = idx - row * C4;
            if (idx >= N_STAGE) break;
            float4 u = v[i].value();
            seen(p0 - halo + row, c4, u);
            if constexpr (PRE_ACT) { u.x = lrelu(u.x); u.y = lrelu(u.y); u.z = lrelu(u.z); u.w = lrelu(u.w); }
            if ((unsigned)(p0 - halo + row) >= (unsigned)valid) u = make_float4(0.f, 0.f, 0.f, 0.f);
            lds_put4<XT>(lds, ((4 * c4 / G::EPL) * STRIDE + row) * G::EPL + 4 * c4 % G::EPL, u);
        }
    }
    __syncthreads();

    const int colbase = wave * (TP / VC_WAVES);
    {
        floatx4 acc[RG][CT];
#pragma unroll
        for (int rg = 0; rg < RG; ++rg)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[rg][ct] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kf = 0; kf < NK; ++kf) {
            uint4 af[RG];
#pragma unroll
            for (int rg = 0; rg < RG; ++rg) {
                af[rg] = ring[kf % AHEAD][rg];
                if (kf + AHEAD < NK) ring[kf % AHEAD][rg] = Wl[((size_t)rg * NK + kf + AHEAD) * 64];
            }
            // this lane's 16 bytes of k: piece q = (tap, channel group); pieces past the end meet zero weights
            const int q = min(kf * 4 + g, NQ - 1);
            const int tap = q / G::GP, cg = q - tap * G::GP;
            const uint4* bl = lds + cg * STRIDE + colbase + n + tap;
            uint4 bv[CT];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) bv[ct] = bl[ct * 16];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int rg = 0; rg < RG; ++rg) acc[rg][ct] = mfma_frag<XT>(af[rg], bv[ct], acc[rg][ct]);
        }
        // ---- epilogue: lane holds rows row0 .. row0 + 3 of column n of every tile
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) {
            const int row0 = (rt0 + rg) * 16 + 4 * g;
            if (row0 >= (EPI == EPI_UP ? ROWS : COUT)) continue;
            if constexpr (EPI == EPI_POST) {
                if (row0 != 0) continue;
                const float b0 = a.bias[0];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const int p = p0 + colbase + ct * 16 + n;
                    if (p < valid) emit(p, tanhf_(acc[rg][ct][0] + b0));
                }
            } else {
                const int co = EPI == EPI_UP ? row0 % COUT : row0;
                const int phase = EPI == EPI_UP ? row0 / COUT : 0;
                const float4 bv = *reinterpret_cast<const float4*>(a.bias + co);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const int p = p0 + colbase + ct * 16 + n;
                    if (p >= valid) continue;
                    const size_t o = ((wbase + p) * U + phase) * COUT + co;
                    const float4 r = make_float4(acc[rg][ct][0] + bv.x, acc[rg][ct][1] + bv.y, acc[rg][ct][2] + bv.z, acc[rg][ct][3] + bv.w);
                    *reinterpret_cast<float4*>(a.out + o) = r;
                }
            }
        }
    }
}

// byte offset of 32 bits from a window's first position: a window is at most (4096 + 16) * 2048 values
template <int CIN> __device__ __forceinline__ float4 quad_at(const float* window, int p, int c4)
{
    return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(window) + (unsigned)(p * CIN + 4 * c4) * 4u);
}

// grid = (tiles of a window, windows, row groups): one convolution of one kind
template <typename XT, int CIN, int ROWS, int COUT, int KS, int EPI, bool PRE_ACT, bool SRC3, int U, bool SHORT, int RG>
__global__ __launch_bounds__(VC_THREADS) void k_vconv(VcArgs a, const int* __restrict__ len, int rate, int window)
{
    constexpr int TP = vc_tp<XT, CIN, ROWS, (KS - 1) / 2, SHORT>();
    __shared__ uint4 lds[vc_stride(TP + 2 * ((KS - 1) / 2)) * VcGeom<XT, CIN>::GP];
    const int w = blockIdx.y, valid = len[w] * rate, p0 = blockIdx.x * TP;
    if (p0 >= valid) return;
    const size_t wbase = (size_t)w * window * rate;
    const float *in0 = a.in0 + wbase * CIN, *in1 = SRC3 ? a.in1 + wbase * CIN : nullptr, *in2 = SRC3 ? a.in2 + wbase * CIN : nullptr;
    auto fetch = [&](int p, int c4) __attribute__((always_inline)) {
        if constexpr (SRC3) return Quad3{quad_at<CIN>(in0, p, c4), quad_at<CIN>(in1, p, c4), quad_at<CIN>(in2, p, c4)};
        else return Quad1{quad_at<CIN>(in0, p, c4)};
    };
    conv_tile<XT, CIN, ROWS, COUT, KS, TP, EPI, PRE_ACT, U, RG>(a, valid, wbase, p0, lds, fetch, [](int, int, float4) {}, [](int, float) {});
}

// The first layer, on the spliced windows [tail(M_pre), M_cur] (Eq. 3 line 1), which exist nowhere else: frames [0, ov) of a window
// with a previous chunk come from the slot's tail, the others from the caller's chunk, four words at a time (his frames need only
// be aligned to them).  Publishes the windows' lengths.  (A launch that wrote the windows to memory first took 2.9 us for one
// window, 4.4 us for 64.)
// The frames that become the slot's tail(M_pre) are kept aside while they are staged, so that this launch is the only one to read the
// caller's frames: his samples, which the last one writes, may lie where they lay.  What the last launch has to know of a window
// lies in device memory then, in one piece (from a list of windows among its own arguments: 8 windows 95.8 us, like this 94.5).  (They wait in `kept`, since other workgroups of this
// launch still read the old tail.  Read once more by workgroups of their own they cost 0.9 us of a round of one window.)
template <typename XT, int RG>
__global__ __launch_bounds__(VC_THREADS) void k_voc_first(VocBatch b, VcArgs a, const float* __restrict__ d_mel, const float* __restrict__ m_tail,
                                                          float* __restrict__ kept, int* __restrict__ len, int4* __restrict__ call, int* __restrict__ turn, int ov, int window,
                                                          Stamps stamps)
{
    constexpr int CIN = VOC_N_MEL, KS = VOC_K_PRE, TP = vc_tp<XT, CIN, VOC_C0, (KS - 1) / 2, true>();
    __shared__ uint4 lds[vc_stride(TP + 2 * ((KS - 1) / 2)) * VcGeom<XT, CIN>::GP];
    const unsigned long long t0 = stamps.now();
    const int w = blockIdx.y, ovw = b.has_prev[w] ? ov : 0, valid = ovw + b.n_frames[w], p0 = blockIdx.x * TP;
    if (p0 >= valid) return;
    const float* mel = d_mel + ((ptrdiff_t)b.src_row[w] - ovw) * CIN;
    const float* tail = m_tail + (size_t)b.slot[w] * ov * CIN;
    auto fetch = [&](int p, int c4) __attribute__((always_inline)) {
        const float* f = (p < ovw ? tail : mel) + p * CIN + 4 * c4;
        return Quad1{make_float4(f[0], f[1], f[2], f[3])};
    };
    // the window's last ov frames, all of them the caller's (where the chunk is the request's last they are kept in vain)
    const int k0 = blockIdx.z == 0 ? max(valid - ov, p0) : valid, k1 = min(valid, p0 + TP);
    auto keep = [&](int p, int c4, float4 v) __attribute__((always_inline)) {
        if (p >= k0 && p < k1) *reinterpret_cast<float4*>(kept + ((size_t)w * ov + p - (valid - ov)) * CIN + 4 * c4) = v;
    };
    conv_tile<XT, CIN, VOC_C0, VOC_C0, KS, TP, EPI_PLAIN, false, 1, RG>(a, valid, (size_t)w * window, p0, lds, fetch, keep, [](int, float) {});
    if (blockIdx.x == 0 && blockIdx.z == 0 && threadIdx.x == 0) {
        const int slot = b.slot[w], mine = turn[slot] ^ 1;
        len[w] = valid;
        turn[slot] = mine;
        call[w] = make_int4(valid, b.out_off[w], slot, mine | (b.has_prev[w] ? VOC_HAS_PREV : 0) | (b.last[w] ? VOC_LAST : 0));
        stamps.begin(t0);
    }
}

// The last layer, and what becomes of its samples S_cur: the first ov * 256 of a window with a previous chunk are fused with the
// slot's tail(S_pre) (Eq. 3 line 2), the response goes to the caller, and the slot's tails become those of this chunk (Eq. 4) unless
// it was the request's last.  Each slot has two tails of audio, which calls read and write in turn (the workgroups of a launch come in
// any order); whose turn it is lies in device memory, where the call's first layer has changed it: a call that was captured goes on
// with the stream at every replay.
// (The mel tail gets its new frames here because the first layer reads the old ones.)  As a launch of its own behind the last layer this took 3.3 us
// for one window, 4.5 us for 64.
template <typename XT, bool SHORT>
__global__ __launch_bounds__(VC_THREADS) void k_voc_last(VcArgs a, const int4* __restrict__ call, const float* __restrict__ alpha, const float* __restrict__ beta,
                                                         float* __restrict__ s_tail, size_t s_tail_turn, float* __restrict__ d_audio,
                                                         const float* __restrict__ kept, float* __restrict__ m_tail, int ov, int window, Stamps stamps)
{
    constexpr int CIN = voc_channels(VOC_STAGES - 1), KS = VOC_K_POST, TP = vc_tp<XT, CIN, 16, (KS - 1) / 2, SHORT>();
    __shared__ uint4 lds[vc_stride(TP + 2 * ((KS - 1) / 2)) * VcGeom<XT, CIN>::GP];
    const int w = blockIdx.y;
    const int4 c = call[w];
    const bool hp = c.w & VOC_HAS_PREV, last = c.w & VOC_LAST, mine = c.w & 1;
    const int valid = c.x * VOC_HOP, p0 = blockIdx.x * TP, N = ov * VOC_HOP;
    if (p0 >= valid) return;
    if (blockIdx.x == 0 && !last) {
        const float* src = kept + w * ov * VOC_N_MEL;
        float* dst = m_tail + (size_t)c.z * ov * VOC_N_MEL;
        for (int e = threadIdx.x; e < ov * VOC_N_MEL; e += VC_THREADS) dst[e] = src[e];
    }
    const size_t slot = (size_t)c.z * N;
    const float* old_tail = s_tail + (mine ? 0 : s_tail_turn) + slot;
    float* new_tail = s_tail + (mine ? s_tail_turn : 0) + slot;
    float* out = d_audio + c.y;
    const int keep = valid - N, n_out = last ? valid : keep;
    auto emit = [&](int i, float v) __attribute__((always_inline)) {
        if (!last && i >= keep) new_tail[i - keep] = v;
        if (i >= n_out) return;
        out[i] = hp && i < N ? alpha[i] * v + beta[i] * old_tail[i] : v;
    };
    const size_t wbase = (size_t)w * window * VOC_HOP;
    const float *in0 = a.in0 + wbase * CIN, *in1 = a.in1 + wbase * CIN, *in2 = a.in2 + wbase * CIN;
    auto fetch = [&](int p, int c4) __attribute__((always_inline)) { return Quad3{quad_at<CIN>(in0, p, c4), quad_at<CIN>(in1, p, c4), quad_at<CIN>(in2, p, c4)}; };
    conv_tile<XT, CIN, 16, 1, KS, TP, EPI_POST, true, 1, 1>(a, valid, wbase, p0, lds, fetch, [](int, int, float4) {}, emit);
    if (threadIdx.x == 0) stamps.end();
}

// ---------------------------------------------------------------------------
// One residual block, all three convolution pairs, on one tile of positions without leaving the CU:
//   for d in (1, 3, 5):  x += conv_{k,1}(lrelu(conv_{k,d}(lrelu(x))))
// The residual stream x of the tile -- TP positions plus the halo H = (k-1)/2 * 12 that the six convolutions
// eat on each side -- stays in registers in the MFMA accumulator layout, so the second convolution of a pair
// accumulates straight onto it.  The operand of the next convolution (leaky ReLU applied, operand type, zero outside
// the request's window) goes through one LDS buffer: written by the lanes that own the values, read as B fragments by
// every wave.  Values near the edge of the region are wrong after a convolution (their neighbours were not staged); the
// error front moves inwards by one halo per convolution and stops exactly at the TP positions that are written out.
// Without HALO the region is a whole window and has no such edge.
//
// A column of the GEMM is a position, and its rows are the channels, where there are 32 or 64 of them.  With 8 or 16
// channels a column is a PAIR of positions, 2 P and 2 P + d for a convolution with dilation d (odd: every position is in
// one pair), and its rows are (position of the pair, channel): the pair shares all but one of its taps at either end, so
// k + 1 taps feed 2 C rows.  Eight channels fill a 16-row tile (half of it was padding), and with sixteen a B fragment
// read from LDS feeds two MFMAs -- k + 1 taps of 16 channels are whole fragments, where k were padded to the same count.
// The operand buffer holds even and odd positions in planes of their own, so the columns of a tap are still consecutive
// rows: 2 P + m d lies in plane m & 1 at row P + (m d - (m & 1)) / 2.
//
// Measured (two-byte mode, windows of 48 frames, one launch): 1 window, 64 / 32 / 16 / 8 channels 34.0 / 13.9 / 9.5 / 9.0 us -> 14.9 / 10.9 /
// 7.8 / 5.4; 64 windows 93.4 / 107 / 70.4 / 119 -> 43.6 / 92 / 59 / 40.  With 32 channels the matrix pipes are busy 36 % of the time and
// the vector units 30 %: a product takes 17 cycles, a vector instruction beside it two to four more, whichever wave of the SIMD it
// is of, and a value costs two and a half of them (leaky ReLU, conversion, store).  One workgroup for a stage's three blocks, with
// their mean stored for the next layer, took as long (352 against 353 us a round of 64); two tiles in a workgroup of eight waves
// that take turns at products and vector work were slower (32 channels 96 -> 102 us).
// ---------------------------------------------------------------------------
struct VrArgs {
    const float* in;                         // the stage's upsampled activations
    float* out;                              // the block's output
    const uint4* W;                          // the six convolutions one after the other, [2 pair + {0: dilated, 1: plain}]
    const float* bias;                       // [2 * VOC_PAIRS][C]
};
struct VrArgs3 {
    VrArgs b[VOC_BLOCKS];
    VocLeast least;                  // the smallest regions
};

constexpr int VR_LDS_MAX = 160 * 1024;

// The weights stream from L1 / L2 into a ring of registers one or two k steps ahead of the products, and on from one convolution into the next: the
// first ones of a convolution are requested behind the last products of the one before.  (Through LDS, as a first version had them, they were a
// quarter to a half of its traffic, and a convolution's 88 KB at 64 channels went through the CU in one burst.  Four steps ahead, with the ring filled
// anew for every convolution, calls of 16 / 64 / 128 windows of 44 frames took 131 / 274 / 481 us, like this 128 / 269 / 469.)  Two operand buffers,
// where LDS holds them, so that one barrier per convolution is enough and a wave that is done prepares the next operand
// while others still read this one.

template <typename XT, int C, int KS, int TP, bool HALO> struct VrGeom {
    using G = VcGeom<XT, C>;
    static constexpr bool PAIR = voc_paired(C);
    // Waves: groups of rows times groups of columns.  Every group of columns fetches the weights of its rows, 16 cycles of the
    // compute unit's L1 a KB: where a region is small they would cost more than the products (64 channels, 128 positions, four
    // groups: 352 KB a convolution of 11 taps, 5600 cycles against 3000), so there the waves share out the rows instead.
    // In the smallest regions, which are mostly halo, a wave has all columns of its rows, so that every one is spared the columns that a
    // convolution's successors do not read any more (TRIM; a call of one window 57.8 -> 56.7 us, fp32, bound by its products, 228 -> 192).
    static constexpr bool TRIM = C == 64 && TP < 64 && HALO;
    static constexpr int THREADS = C == 64 && !TRIM ? 512 : 256;
    static constexpr int RGROUPS = C == 64 ? (TP < 128 ? 4 : 2) : C == 32 && TP < 128 ? 2 : 1;
    static constexpr int CGROUPS = THREADS / 64 / RGROUPS;
    static constexpr int HALF = (KS - 1) / 2;
    static constexpr int H = HALO ? HALF * 12 : 0;            // sum over d = 1, 3, 5 of (d + 1) * HALF
    static constexpr int H_MOST = HALO ? (voc_block_k(VOC_BLOCKS - 1) - 1) / 2 * 12 : 0;
    static constexpr int PW = PAIR ? 32 : 16;                 // positions per column tile
    static constexpr int NCOL = (TP + 2 * H_MOST + CGROUPS * PW - 1) / (CGROUPS * PW);  // column tiles per wave
    static constexpr int W = CGROUPS * PW * NCOL;             // positions of the region
    // ... of which so many come out right: TP or a little more with the longest kernel, more with the others, whose halo is shorter.  (With
    // TP of them in every block, 128 windows of 44 frames 481 us, like this 473)
    static constexpr int OUT = HALO ? W - 2 * H : TP;
    // column tiles of convolution i's output that are read again: [first, end)
    __device__ static constexpr int edge(int i) { return i < 0 ? 0 : edge(i - 1) + HALF * (i & 1 ? 1 : i + 1); }      // i even: dilation i + 1
    __device__ static constexpr int first(int i) { return TRIM ? edge(i) / 16 : 0; }
    __device__ static constexpr int end(int i) { return TRIM ? (W - edge(i) + 15) / 16 : NCOL; }
    static_assert(!TRIM || (CGROUPS == 1 && !PAIR), "a wave's columns are the region's");
    static constexpr int RT = (PAIR ? 2 * C : C) / 16 / RGROUPS;          // row tiles per wave
    static constexpr int TAPS = PAIR ? KS + 1 : KS;
    static constexpr int NK = TAPS * C / Frag<XT>::KB;
    // (ten products a k step are 160 cycles: with two steps ahead there 128 windows 464 -> 472 us, with one where there are fewer products 32
    // windows 165.8 -> 169.2)
    static constexpr int AHEAD = TRIM ? 2 : RT * NCOL >= 10 || NK == 1 ? 1 : 2;
    static_assert(2 * NK % AHEAD == 0, "two convolutions go round the ring in whole turns");
    // zero rows on each side: the widest tap offset
    static constexpr int PAD = PAIR ? (5 * (HALF + 1) + 1) / 2 : 5 * HALF;
    static constexpr int PLANE = (PAIR ? W / 2 : W) + 2 * PAD;            // rows of a plane
    // 16-byte pieces: a plane per 16 bytes of channels, and of even and odd positions.  Lanes l and l + 16 of a B fragment read
    // the same rows (or, with 8 channels, rows of even and odd positions up to three apart) of different planes: LDS gives 256
    // bytes a cycle where their distance is a multiple of 16 pieces, half of that otherwise (4.4 and 8.0 cycles a wave's read)
    static constexpr int EVEN = PAIR ? (PLANE + 2 + 15) / 16 * 16 : 0;    // where the even positions begin, up to a shift
    static constexpr int STRIDE = (EVEN + PLANE + 15) / 16 * 16;          // between channel planes
    static constexpr int OPERAND_VECS = STRIDE * G::GP;
    static constexpr bool TWO = 2 * OPERAND_VECS * 16 + 2 * VOC_PAIRS * C * 4 <= VR_LDS_MAX;
    static constexpr int BIAS_AT = (TWO ? 2 : 1) * OPERAND_VECS;         // the six biases
    static constexpr int BYTES = BIAS_AT * 16 + 2 * VOC_PAIRS * C * 4;
    static constexpr int W_BYTES = RT * RGROUPS * NK * 1024;             // weights of one convolution
    static_assert(RT * RGROUPS * 16 == (PAIR ? 2 * C : C) && NK * Frag<XT>::KB == TAPS * C, "whole tiles and fragments");
    // first piece of the plane of position parity s.  With 8 channels neighbouring taps of a dilation d lie (d + 1) / 2 rows apart in the
    // odd and the even plane: the shift is that of d = 1 in the second buffer and of d = 3 in the first, which has d = 1, 3, 5 in turn
    __device__ static constexpr int plane(int s, int buf) { return !PAIR || s ? 0 : EVEN - (TWO && buf == 0 ? 2 : 1); }
    static_assert(HALO || !PAIR, "a pair's second position is missing at the region's first positions: they have to lie in a halo");
};

// The weights of a block's six convolutions in A-fragment order: a fragment's place is a scalar offset, so all of them share one
// address register, and no pointer has to be loaded before a convolution's first fragment can be requested.
template <typename R> struct VrWeights {
    __amdgpu_buffer_rsrc_t rsrc;
    int rt0, lane;
    __device__ __forceinline__ VrWeights(const uint4* W, int rt0, int lane)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(W), 0, 2 * VOC_PAIRS * R::W_BYTES, BUFFER_RSRC_RAW)), rt0(rt0), lane(lane) {}
    __device__ __forceinline__ uint4 at(int conv, int rt, int kf) const
    {
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, conv * R::W_BYTES + ((rt0 + rt) * R::NK + kf) * 1024, 0);
        return make_uint4(v.x, v.y, v.z, v.w);
    }
};
template <int N> struct Int {
    static constexpr int value = N;
    __device__ constexpr operator int() const { return N; }
};
template <typename R> using VrRing = uint4[R::AHEAD][R::RT];
template <typename R> __device__ __forceinline__ void ring_fill(VrRing<R>& ring, const VrWeights<R>& W)
{
#pragma unroll
    for (int kf = 0; kf < R::AHEAD; ++kf)
#pragma unroll
        for (int rt = 0; rt < R::RT; ++rt) ring[kf][rt] = W.at(0, rt, kf);
}

// acc += W * operand, or bias + W * operand (INIT), for the wave's column tiles CT0 .. CT1 - 1.  A k step's B fragments are requested before the
// products of the step before.
template <typename XT, typename R, bool INIT, int CT0, int CT1>
__device__ __forceinline__ void conv_regs(const VrWeights<R>& W, int conv, VrRing<R>& ring, int dil, const uint4* lds, int buf, int col0, int lane,
                                          const floatx4 (&bias)[R::RT], floatx4 (&acc)[R::RT][R::NCOL])
{
    using G = typename R::G;
    constexpr int NK = R::NK, RT = R::RT, NCOL = R::NCOL, GP = G::GP;
    const int n = lane & 15, g = lane >> 4, next = min(conv + 1, 2 * VOC_PAIRS - 1);      // (the last one's request is dropped)
    // this lane's 16 bytes of k in fragment kf: piece 4 kf + g = (tap, channel group)
    auto b_at = [&](int kf) __attribute__((always_inline)) {
        constexpr int STEP = GP < 4 ? 4 / GP : 1;             // taps per fragment
        if constexpr (R::PAIR && STEP % 2 == 0) {             // the parity of a lane's tap does not change from fragment to fragment
            const int m = g / GP - R::HALF, pl = m & 1;
            return (g % GP) * R::STRIDE + R::plane(pl, buf) + R::PAD + col0 + n + ((m * dil - pl) >> 1) + kf * (STEP / 2) * dil;
        } else {
            const int q = 4 * kf + g, m = q / GP - R::HALF;
            if constexpr (R::PAIR) return (q % GP) * R::STRIDE + R::plane(m & 1, buf) + R::PAD + col0 + n + ((m * dil - (m & 1)) >> 1);
            else return (q % GP) * R::STRIDE + R::PAD + col0 + n + m * dil;
        }
    };
    uint4 bv[2][NCOL];
    auto request = [&](int kf) __attribute__((always_inline)) {
        const uint4* bl = lds + b_at(kf);
#pragma unroll
        for (int ct = CT0; ct < CT1; ++ct) bv[kf & 1][ct] = bl[ct * 16];
    };
    request(0);
#pragma unroll
    for (int kf = 0; kf < NK; ++kf) {
        uint4 af[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            constexpr int PHASE = INIT ? 0 : NK % R::AHEAD;
            uint4& r = ring[(kf + PHASE) % R::AHEAD][rt];
            af[rt] = r;
            r = kf + R::AHEAD < NK ? W.at(conv, rt, kf + R::AHEAD) : W.at(next, rt, kf + R::AHEAD - NK);
        }
        if (kf + 1 < NK) request(kf + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ct = CT0; ct < CT1; ++ct)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt][ct] = mfma_frag<XT>(af[rt], bv[kf & 1][ct], INIT && kf == 0 ? bias[rt] : acc[rt][ct]);
    }
}

template <typename XT, int C, int KS, int TP, bool HALO>
__device__ __forceinline__ void resblock_tile(const VrArgs& a, int valid, size_t wbase, int tile, uint4* lds)
{
    using R = VrGeom<XT, C, KS, TP, HALO>;
    const int p0 = tile * R::OUT;
    if (p0 >= valid) return;
    using G = typename R::G;
    constexpr int RT = R::RT, NCOL = R::NCOL;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int col0 = wave % R::CGROUPS * 16 * NCOL;            // this wave's first column of the region
    const int rt0 = wave / R::CGROUPS * RT;                    // ... and its first row tile
    const int pbase = p0 - R::H;                 // the region's first position inside the window
    // the lane's four rows of row tile rt: position s of the pair, channels ch .. ch + 3
    auto part = [&](int rt) __attribute__((always_inline)) { return !R::PAIR ? 0 : C == 8 ? g >> 1 : rt; };
    auto chan = [&](int rt) __attribute__((always_inline)) { return R::PAIR ? (C == 8 ? 4 * (g & 1) : 4 * g) : (rt0 + rt) * 16 + 4 * g; };
    // position inside the region of row tile rt, column tile ct, in a layout whose pairs are d apart.  c = this lane's column of
    // column tile 0, made anew by its users: positions kept from one phase to the next would cost more registers than the sums
    auto column = [&]() __attribute__((always_inline)) {
        int c = col0 + n;
        asm volatile("" : "+v"(c));
        return c;
    };
    auto pos = [&](int c, int rt, int ct, int d) __attribute__((always_inline)) {
        const int col = c + ct * 16;
        return R::PAIR ? 2 * col + part(rt) * d : col;
    };
    // byte offsets of 32 bits from the window's first position: a window is at most (4096 + 16) * 2048 values
    const char* in = reinterpret_cast<const char*>(a.in + wbase * C);
    char* out = reinterpret_cast<char*>(a.out + wbase * C);
    auto byte_at = [&](int p, int rt) __attribute__((always_inline)) { return (unsigned)(p * C + chan(rt)) * 4u; };

    const VrWeights<R> weights(a.W, rt0, lane);
    VrRing<R> ring;
    float* const lds_bias = reinterpret_cast<float*>(lds + R::BIAS_AT);
    floatx4 x[RT][NCOL];
    {
        const int c = column();
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < NCOL; ++ct) {                 // clamped: what lies outside the window is never put in the buffer
                const int p = min(max(pbase + pos(c, rt, ct, 1), 0), valid - 1);
                x[rt][ct] = *reinterpret_cast<const floatx4*>(in + byte_at(p, rt));
            }
    }
    ring_fill<R>(ring, weights);
    for (int i = tid; i < 2 * VOC_PAIRS * C; i += R::THREADS) lds_bias[i] = a.bias[i];
    // Rows in front of and behind the region, and those of positions outside the window, are zero: nothing but a pair's second
    // position a little past the region's end is ever stored there.
    const int r0 = max(-pbase, 0), r1 = min(valid - pbase, R::W);         // positions r0 .. r1 - 1 of the region exist
    const bool edge = r0 > 0 || r1 < R::W;
    auto zero_rows = [&](uint4* plane, int from, int to) __attribute__((always_inline)) {
        for (int row = from + tid; row < to; row += R::THREADS)
#pragma unroll
            for (int cg = 0; cg < G::GP; ++cg) plane[cg * R::STRIDE + row] = make_uint4(0, 0, 0, 0);
    };
#pragma unroll
    for (int buf = 0; buf < (R::TWO ? 2 : 1); ++buf)
#pragma unroll
        for (int pl = 0; pl < (R::PAIR ? 2 : 1); ++pl) {       // row PAD + i of plane pl: position 2 i + pl, or i
            uint4* plane = lds + buf * R::OPERAND_VECS + R::plane(pl, buf);
            zero_rows(plane, 0, R::PAD + (R::PAIR ? (r0 - pl + 1) >> 1 : r0));
            zero_rows(plane, R::PAD + (R::PAIR ? (r1 - pl + 1) >> 1 : r1), R::PLANE);
        }
    // operand of the next convolution: lrelu, operand type, positions of the window only; v in the layout of pairs d apart; column tiles as above
    auto put = [&](uint4* at, int buf, const floatx4 (&v)[RT][NCOL], int d, auto ct0, auto ct1) __attribute__((always_inline)) {
        const int c = column();
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int ch = chan(rt), s = part(rt);
            const int e = ((ch / G::EPL) * R::STRIDE + (s ? R::plane(1, buf) : R::plane(0, buf)) + s * ((d - 1) >> 1) + R::PAD + c) * G::EPL + ch % G::EPL;
            auto store = [&](int ct) __attribute__((always_inline)) {
                const floatx4 f = v[rt][ct];
                lds_put4<XT>(at, e + ct * 16 * G::EPL, make_float4(lrelu(f[0]), lrelu(f[1]), lrelu(f[2]), lrelu(f[3])));
            };
            if (edge) {
#pragma unroll
                for (int ct = ct0; ct < ct1; ++ct)
                    if ((unsigned)(pbase + pos(c, rt, ct, d)) < (unsigned)valid) store(ct);
            } else {
#pragma unroll
                for (int ct = ct0; ct < ct1; ++ct) store(ct);
            }
        }
    };
    auto biases = [&](int conv, floatx4 (&v)[RT]) __attribute__((always_inline)) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) v[rt] = *reinterpret_cast<const floatx4*>(lds_bias + conv * C + chan(rt));
    };
    uint4* const lds1 = lds + (R::TWO ? R::OPERAND_VECS : 0);
    put(lds, 0, x, 1, Int<0>{}, Int<NCOL>{});
    lds_barrier();
    auto do_pair = [&](int pair, auto trim) __attribute__((always_inline)) {       // trim: the pair's number where its columns depend on it
        constexpr int P = decltype(trim)::value, A0 = R::first(2 * P), A1 = R::end(2 * P), B0 = R::first(2 * P + 1), B1 = R::end(2 * P + 1);
        const int d = 2 * pair + 1;
        floatx4 t[RT][NCOL], b[RT];
        biases(2 * pair, b);
        conv_regs<XT, R, true, A0, A1>(weights, 2 * pair, ring, d, lds, 0, col0, lane, b, t);
        if constexpr (!R::TWO) lds_barrier();     // every wave has read the old operand
        __builtin_amdgcn_s_setprio(2);            // vector work goes ahead of the products of the wave it shares a SIMD with
        put(lds1, 1, t, d, Int<A0>{}, Int<A1>{});
        __builtin_amdgcn_s_setprio(0);
        biases(2 * pair + 1, b);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = B0; ct < B1; ++ct) x[rt][ct] += b[rt];
        lds_barrier();
        conv_regs<XT, R, false, B0, B1>(weights, 2 * pair + 1, ring, 1, lds1, 1, col0, lane, b, x);
        if (pair + 1 < VOC_PAIRS) {
            if constexpr (!R::TWO) lds_barrier();
            __builtin_amdgcn_s_setprio(2);
            put(lds, 0, x, 1, Int<B0>{}, Int<B1>{});
            __builtin_amdgcn_s_setprio(0);
            lds_barrier();
        }
    };
    if constexpr (R::TRIM) {
        static_assert(VOC_PAIRS == 3, "the pairs one by one");
        do_pair(0, Int<0>{});
        do_pair(1, Int<1>{});
        do_pair(2, Int<2>{});
    } else {
#pragma unroll 1
        for (int pair = 0; pair < VOC_PAIRS; ++pair) do_pair(pair, Int<0>{});
    }
    const int o0 = R::H, o1 = min(R::H + R::OUT, valid - pbase);  // positions of the region that are this tile's output
    const int c = column();
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < NCOL; ++ct) {
            const int j = pos(c, rt, ct, 1);
            if (j >= o0 && j < o1) *reinterpret_cast<floatx4*>(out + byte_at(pbase + j, rt)) = x[rt][ct];
        }
}

// The three residual blocks (kernels 3, 7, 11) of a stage: grid = (tiles, windows, 3), the longest first.  The smallest regions: one dimension, the
// regions of all windows (VocLeast).
template <typename XT, int C, int TP, bool HALO>
__global__ __launch_bounds__((VrGeom<XT, C, 3, TP, HALO>::THREADS), C == 8 ? (sizeof(XT) == 2 ? 4 : 3) : 2) void k_vres(VrArgs3 a3, const int* __restrict__ len, int rate, int window)
{
    extern __shared__ uint4 lds_dyn[];
    int w = blockIdx.y, block = VOC_BLOCKS - 1 - blockIdx.z, tile = blockIdx.x;
    if constexpr (VrGeom<XT, C, 3, TP, HALO>::TRIM) block = a3.least.block(blockIdx.x, &w, &tile);
    const int valid = len[w] * rate;
    const size_t wbase = (size_t)w * window * rate;
    if (block == 0) resblock_tile<XT, C, 3, TP, HALO>(a3.b[0], valid, wbase, tile, lds_dyn);
    else if (block == 1) resblock_tile<XT, C, 7, TP, HALO>(a3.b[1], valid, wbase, tile, lds_dyn);
    else resblock_tile<XT, C, 11, TP, HALO>(a3.b[2], valid, wbase, tile, lds_dyn);
}

// What a call asks of every launch: its windows, the frames of the longest one and of all.
struct Load {
    int n, longest, frames;
};

// grid = (tiles of a window, windows, row groups).  SHORT: tiles of 64 positions - for the layer that runs at one position
// per frame, where a window is a few dozen positions long, and for every layer of a batch so small that the large tiles
// would leave most of the chip idle (an output's sum does not depend on the tile it falls in).
// (Calls of 48 / 64 / 128 windows with the line at 512 workgroups 226 / 270.3 / 480.9 us, at 1024 220 / 266.4 / 479.7, at 2048 220 / 266 / 475.)
constexpr int VC_SHORT_BELOW = 2048;             // workgroups of the large tiling below which the short one is used
// Row tiles per workgroup: four, or one where that is at most two workgroups for every compute unit: all its weights are on their way then before the
// positions are staged (calls of 1 / 4 / 8 windows 62.3 / 81.6 / 99.7 -> 57.7 / 77.7 / 95.8 us; fp32 242.7 / 347 / 418 -> 228.7 / 336 / 405; with the
// line at one workgroup 4 / 16 / 40 windows take 1 / 1 / 2 us longer).
constexpr int VC_FEW = 512;
template <typename XT, int CIN, int ROWS, int COUT, int KS, int EPI, bool PRE_ACT, bool SRC3, int U, bool SHORT>
void conv_launch(const VcArgs& a, const int* len, int rate, int window, Load c, hipStream_t s)
{
    constexpr int TP = vc_tp<XT, CIN, ROWS, (KS - 1) / 2, SHORT>();
    constexpr int RT = ROWS / 16, RG = RT < 4 ? RT : 4;
    const dim3 grid((c.longest * rate + TP - 1) / TP, c.n, RT / RG);
    if constexpr (!SHORT) {
        if ((long)grid.x * grid.y * grid.z < VC_SHORT_BELOW) {
            conv_launch<XT, CIN, ROWS, COUT, KS, EPI, PRE_ACT, SRC3, U, true>(a, len, rate, window, c, s);
            return;
        }
    }
    if constexpr (SHORT && RG > 1)
        if ((long)grid.x * grid.y * RT <= VC_FEW) {
            hipLaunchKernelGGL((k_vconv<XT, CIN, ROWS, COUT, KS, EPI, PRE_ACT, SRC3, U, SHORT, 1>), dim3(grid.x, grid.y, RT), dim3(VC_THREADS), 0, s, a, len, rate, window);
            return;
        }
    hipLaunchKernelGGL((k_vconv<XT, CIN, ROWS, COUT, KS, EPI, PRE_ACT, SRC3, U, SHORT, RG>), grid, dim3(VC_THREADS), 0, s, a, len, rate, window);
}

template <typename XT, int C, int TP, bool HALO>
hipError_t blocks_launch_tp(const VrArgs3& a, const int* len, int rate, int window, Load c, hipStream_t s)
{
    constexpr int L3 = VrGeom<XT, C, 3, TP, HALO>::BYTES, L7 = VrGeom<XT, C, 7, TP, HALO>::BYTES, L11 = VrGeom<XT, C, 11, TP, HALO>::BYTES;
    constexpr int LDS = L3 > L7 ? (L3 > L11 ? L3 : L11) : (L7 > L11 ? L7 : L11);      // the three kernels share a launch
    auto kern = k_vres<XT, C, TP, HALO>;
    static bool attr_set = false;                            // dynamic LDS above 64 KB has to be allowed once per kernel
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    constexpr int OUT = VrGeom<XT, C, voc_block_k(VOC_BLOCKS - 1), TP, HALO>::OUT;       // (the others have as many tiles or fewer)
    dim3 grid(HALO ? (c.longest * rate + OUT - 1) / OUT : 1, c.n, VOC_BLOCKS);
    VrArgs3 args = a;
    if constexpr (VrGeom<XT, C, 3, TP, HALO>::TRIM) {
        static_assert(VrGeom<XT, C, 3, TP, HALO>::OUT == voc_least_out(0) && VrGeom<XT, C, 7, TP, HALO>::OUT == voc_least_out(1) && OUT == voc_least_out(2), "what comes out right");
        args.least = voc_least(c.n, c.longest * rate);
        grid = dim3(args.least.all());
    }
    hipLaunchKernelGGL(kern, grid, dim3(VrGeom<XT, C, 3, TP, HALO>::THREADS), LDS, s, args, len, rate, window);
    return hipSuccess;
}

// Positions per workgroup of the tilings: small batches take half of the large tiles, a request or two a quarter -- more
// workgroups, each with a shorter chain, and a larger share of halo.  Behind the longest halo (120) a region is a whole number of
// column tiles.  With 64 channels, where a window is a few hundred positions and a region's products are the longest, a
// request alone takes the smallest region there is.
template <int C, int LEVEL> constexpr int vr_tp() { return LEVEL == 3 ? 8 : ((C >= 32 ? 256 : 512) >> LEVEL) + 8; }
// With 64 channels (8 positions a frame) the halo of a tile of 128 doubles its work.  A window of up to 384 positions fits a workgroup's
// registers and LDS whole and needs none: a CU per window and block, which pays where there are enough of them, unless half a tile holds the window.
//
// All lines below look at the call's longest window, whatever the configuration allows: `large` counts positions in large tiles, the others their own
// workgroups.  (By the configured window, 44 frames: calls of 4 / 16 / 64 / 128 windows of 12 frames 62.6 / 85.9 / 152 / 204 us, like this 58.5 / 79.1 /
// 135 / 189; fp32 225 / 357 / 781 / 1100 -> 197 / 250 / 584 / 881; of 28 frames 66.7 / 107 / 202 / 330 -> 64.1 / 105 / 198 / 327, fp32 229 / 457 / 1095 / 1743 -> 222 / 428 / 934 / 1689.)
// Us a call of n windows of 44 frames unless said otherwise, on one side of each line and on the other:
//   whole       tiles / whole: 40, 48, 64, 96 windows 195 / 198, 221 / 219, 270 / 263, 377 / 357, of 28 frames 48, 64, 96: 164 / 172, 198 / 199, 275 / 257; fp32 48, 64:
//               1138 / 1198, 1475 / 1435, of 28 frames 64, 96: 933 / 1050, 1400 / 1366; of 12 frames half a tile holds them: 96 windows 159 / 169, fp32 800 / 864
//   smallest    next larger / smallest: 3, 4 windows 77 / 72, 80 / 76, 5, 8: 89 / 87, 98 / 100 (beyond the line); fp32 4, 8: 337 / 244, 409 / 400, 10, 12: 428 / 439, 472 / 546
//   quarter     half / quarter: 24, 28 windows 148 / 146, 159 / 163; fp32 24, 32, 36: 709 / 651, 826 / 821, 892 / 948; of 48 frames 28, 32: 780 / 776, 844 / 902;
//               of 68 frames 20, 24: 787 / 781, 895 / 954 (beyond VR_TINY_FULL); 4 fp32 windows of up to 400 frames, which have quarters without work, 653 / 592
//   half        large / half: 24, 28 windows 146.0 / 149.2, 157.1 / 159.2; fp32 707 / 734, 762 / 806
constexpr int VR_WHOLE = 384;
template <typename XT> constexpr int vr_whole_from() { return sizeof(XT) == 4 ? 224 : 192; }
constexpr int VR_SMALL_BELOW = 700;
template <typename XT, int C> constexpr int vr_tiny_upto() { return C != 64 ? 470 : sizeof(XT) == 4 ? 576 : 360; }
constexpr int VR_TINY_FULL = 490;                // quarters' worth of positions, of all windows together
template <typename XT> constexpr int vr_least_upto() { return sizeof(XT) == 4 ? 1100 : 800; }

template <typename XT, int C>
hipError_t blocks_launch(const VrArgs3& a, const int* len, int rate, int window, Load c, hipStream_t s)
{
    const long positions = (long)c.longest * rate, regions = (long)c.n * VOC_BLOCKS, large = positions * regions / vr_tp<C, 0>();
    auto tiles = [&](int tp) { return (positions + tp - 1) / tp * regions; };
    if constexpr (C == 64) {
        if (positions <= VR_WHOLE && positions > vr_tp<C, 1>() && large >= vr_whole_from<XT>()) return blocks_launch_tp<XT, C, VR_WHOLE, false>(a, len, rate, window, c, s);
        if (tiles(vr_tp<C, 3>()) <= vr_least_upto<XT>()) return blocks_launch_tp<XT, C, vr_tp<C, 3>(), true>(a, len, rate, window, c, s);
    }
    if (tiles(vr_tp<C, 2>()) <= vr_tiny_upto<XT, C>() && (long)c.frames * rate * VOC_BLOCKS / vr_tp<C, 2>() <= VR_TINY_FULL) return blocks_launch_tp<XT, C, vr_tp<C, 2>(), true>(a, len, rate, window, c, s);
    return large < VR_SMALL_BELOW ? blocks_launch_tp<XT, C, vr_tp<C, 1>(), true>(a, len, rate, window, c, s)
                                  : blocks_launch_tp<XT, C, vr_tp<C, 0>(), true>(a, len, rate, window, c, s);
}

template <typename XT, int S>
hipError_t stage_launch(const VocoderPtrs& d, Load c, hipStream_t s)
{
    constexpr int CIN = VOC_C0 >> S, C = CIN / 2, U = voc_rate(S);
    constexpr int rate_in = S == 0 ? 1 : voc_cum_rate(S - 1), rate = voc_cum_rate(S);
    VcArgs up{};
    up.in0 = S == 0 ? d.x0 : d.r[0];
    up.in1 = d.r[1];
    up.in2 = d.r[2];
    up.out = d.y;
    up.W = reinterpret_cast<const uint4*>(d.up_w[S]);
    up.bias = d.up_b[S];
    conv_launch<XT, CIN, U * C, C, 3, EPI_UP, true, (S > 0), U, (S == 0)>(up, d.len, rate_in, d.window, c, s);
    VrArgs3 rb{};
    for (int b = 0; b < VOC_BLOCKS; ++b) {
        rb.b[b].in = d.y;
        rb.b[b].out = d.r[b];
        rb.b[b].W = reinterpret_cast<const uint4*>(d.res_w[S][b]);
        rb.b[b].bias = d.res_b[S][b];
    }
    return blocks_launch<XT, C>(rb, d.len, rate, d.window, c, s);
}

template <typename XT>
hipError_t vocoder_typed(const VocoderPtrs& d, const VocBatch& b, const float* d_mel, float* d_audio, hipStream_t s)
{
    Load c{b.n, 0, 0};
    for (int w = 0; w < b.n; ++w) {
        const int f = (b.has_prev[w] ? d.overlap : 0) + b.n_frames[w];
        c.longest = std::max(c.longest, f);
        c.frames += f;
    }
    VcArgs pre{};
    pre.out = d.x0;
    pre.W = reinterpret_cast<const uint4*>(d.pre_w);
    pre.bias = d.pre_b;
    constexpr int PRE_TP = vc_tp<XT, VOC_N_MEL, VOC_C0, (VOC_K_PRE - 1) / 2, true>();
    const int pre_tiles = (c.longest + PRE_TP - 1) / PRE_TP;
    auto first = [&](auto kern, int row_groups) {
        hipLaunchKernelGGL(kern, dim3(pre_tiles, b.n, row_groups), dim3(VC_THREADS), 0, s, b, pre, d_mel, d.m_tail, d.kept, d.len, d.call, d.turn, d.overlap, d.window, d.stamps);
    };
    if ((long)pre_tiles * b.n * (VOC_C0 / 16) <= VC_FEW) first(k_voc_first<XT, 1>, VOC_C0 / 16);
    else first(k_voc_first<XT, 4>, VOC_C0 / 64);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = stage_launch<XT, 0>(d, c, s);
    if (e == hipSuccess) e = stage_launch<XT, 1>(d, c, s);
    if (e == hipSuccess) e = stage_launch<XT, 2>(d, c, s);
    if (e == hipSuccess) e = stage_launch<XT, 3>(d, c, s);
    if (e != hipSuccess) return e;
    VcArgs post{};
    post.in0 = d.r[0];
    post.in1 = d.r[1];
    post.in2 = d.r[2];
    post.W = reinterpret_cast<const uint4*>(d.post_w);
    post.bias = d.post_b;
    auto last = [&](auto kern, int tp) {
        hipLaunchKernelGGL(kern, dim3((c.longest * VOC_HOP + tp - 1) / tp, b.n), dim3(VC_THREADS), 0, s, post, d.call, d.alpha, d.beta, d.s_tail, d.s_tail_turn, d_audio,
                           d.kept, d.m_tail, d.overlap, d.window, d.stamps);
    };
    constexpr int CL = voc_channels(VOC_STAGES - 1), LONG_TP = vc_tp<XT, CL, 16, (VOC_K_POST - 1) / 2>(), SHORT_TP = vc_tp<XT, CL, 16, (VOC_K_POST - 1) / 2, true>();
    if ((long)((c.longest * VOC_HOP + LONG_TP - 1) / LONG_TP) * b.n < VC_SHORT_BELOW) last(k_voc_last<XT, true>, SHORT_TP);
    else last(k_voc_last<XT, false>, LONG_TP);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_vocoder(const VocoderPtrs& d, int wdtype, const VocBatch& b, const float* d_mel, float* d_audio, hipStream_t s)
{
    return wdtype == 0 ? vocoder_typed<float>(d, b, d_mel, d_audio, s) : vocoder_typed<h16_t>(d, b, d_mel, d_audio, s);
}

}  // namespace tts
