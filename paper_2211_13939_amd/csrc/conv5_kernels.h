// Kernel-5 convolution over time on a ragged batch of windows, on MFMA: shared by the PostNet (windows = chunks with
// context, tanh) and the acoustic encoder (windows = the token sequences of requests, ReLU).
//
// A convolution layer is a GEMM  Y[c_out][column] = W[c_out][tap * C_in + c_in] * X[c_in][column + tap - 2]
// with the columns of all windows packed back to back; a column that would leave its own window
// reads zero ("same" padding per window).  It runs on MFMA with 16 columns as N:
//   * activations between layers live in HBM in the same MFMA B-operand fragment order as the
//     decoder's activations (16 columns form a tile, 64 bytes of channels per fragment), so a
//     layer's output is stored exactly as the next layer loads it;
//   * a workgroup owns one 16-row tile of output channels and one or two column tiles; it stages the
//     columns it needs (its tiles plus two columns on either side) in LDS once, and its eight
//     waves split K = 5 * C_in: every wave keeps its share of the weight fragments in registers,
//     builds the five shifted B operands from LDS, and the partial sums meet in LDS;
//   * bias, the activation, the residual sum of the PostNet's last layer and the selection of the chunk's own
//     frames are fused into the epilogue.
#pragma once
#include "postnet_kernels.h"
#include "mfma.h"

namespace tts {

constexpr int PN_THREADS = 512;
constexpr int PN_WAVES = PN_THREADS / 64;
constexpr int PN_HALO = PN_TAPS / 2;             // columns needed on either side of a tile
// column tiles per workgroup: what fits 64 KB of LDS next to the reduction buffer
template <typename XT> struct PnCT { static constexpr int value = sizeof(XT) == 2 ? 2 : 1; };

// epilogue of a layer: tanh / ReLU into the next layer's input, or the PostNet's last layer
enum { PN_EPI_TANH = 0, PN_EPI_LAST = 1, PN_EPI_RELU = 2 };
template <int EPI> __device__ __forceinline__ float pn_act(float x) { return EPI == PN_EPI_RELU ? fmaxf(x, 0.f) : tanhf_(x); }

// One layer.  grid = (COUT / 16, ceil(column tiles / PnCT)).
//   cmeta[col] = (frames in the column's window << 16) | the column's index inside its window
//   PN_EPI_LAST: out[orow[col]][*] = mel[col][*] + bias + sum  for columns with orow >= 0 (the chunk's own frames)
template <typename XT, int CIN, int COUT, int EPI>
__global__ __launch_bounds__(PN_THREADS) void k_pn_conv(
    const uint4* __restrict__ Wfrag, const float* __restrict__ bias, const uint4* __restrict__ Xin, XT* __restrict__ Xout,
    const int* __restrict__ cmeta, int n_ctiles, const float* __restrict__ mel, int n_mel, const int* __restrict__ orow,
    float* __restrict__ out, Stamps stamps)
{
    constexpr int KB = Frag<XT>::KB, EPL = Frag<XT>::EPL;
    constexpr int PN_CT = PnCT<XT>::value;
    constexpr int NKF = CIN / KB;                      // channel fragments per column tile
    constexpr int NKT = PN_TAPS * NKF;                 // K fragments of the GEMM
    constexpr int NFW = (NKT + PN_WAVES - 1) / PN_WAVES;   // per wave
    constexpr int ROWS = PN_CT * 16 + 2 * PN_HALO;     // staged columns
    constexpr int LD = CIN * (int)sizeof(XT) + 16;     // bytes per staged column: an odd number of 16-byte pieces
    static_assert(CIN % KB == 0 && COUT % 16 == 0, "channel counts must fill whole fragments / row tiles");

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int jl = lane & 15, g = lane >> 4;
    const int rt = blockIdx.x;
    const int ct0 = blockIdx.y * PN_CT;

    __shared__ __attribute__((aligned(16))) unsigned char s_x[ROWS * LD];
    __shared__ floatx4 red[PN_WAVES][PN_CT][64];

    // this wave's share of the weights: fragments wave, wave + 8, ... of row tile rt (k = tap * CIN + channel)
    uint4 a[NFW];
#pragma unroll
    for (int i = 0; i < NFW; ++i) {
        const int f = wave + i * PN_WAVES;
        a[i] = f < NKT ? Wfrag[xfrag(NKT, rt, f, lane)] : make_uint4(0, 0, 0, 0);
    }
    // the columns of this workgroup's tiles and two more on either side, once, into LDS:
    // piece (row, channel fragment cf, lane group gg) = 16 bytes of channels cf * KB + gg * EPL ..
    const int col_first = ct0 * 16 - PN_HALO;
    const int n_col_pad = n_ctiles * 16;
    for (int p = tid; p < ROWS * NKF * 4; p += PN_THREADS) {
        const int row = p / (NKF * 4), rem = p - row * (NKF * 4);
        const int cf = rem >> 2, gg = rem & 3;
        const int col = col_first + row;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (col >= 0 && col < n_col_pad) v = Xin[xfrag(NKF, col >> 4, cf, (col & 15) + 16 * gg)];
        *reinterpret_cast<uint4*>(&s_x[row * LD + (cf * KB + gg * EPL) * (int)sizeof(XT)]) = v;
    }
    // which taps stay inside the column's own window (bit d+2 for column offset d)
    int tapmask[PN_CT];
#pragma unroll
    for (int c = 0; c < PN_CT; ++c) {
        const int col = min((ct0 + c) * 16 + jl, n_col_pad - 1);
        const int m = cmeta[col];
        const int t = m & 0xFFFF, T = m >> 16;
        int bits = 0;
#pragma unroll
        for (int d = -PN_HALO; d <= PN_HALO; ++d) bits |= (t + d >= 0 && t + d < T) ? (1 << (d + PN_HALO)) : 0;
        tapmask[c] = bits;
    }
    floatx4 bias4 = {0.f, 0.f, 0.f, 0.f};
    if (wave < PN_CT) bias4 = *reinterpret_cast<const floatx4*>(bias + rt * 16 + 4 * g);
    __syncthreads();

#pragma unroll
    for (int c = 0; c < PN_CT; ++c) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        if (ct0 + c < n_ctiles) {
#pragma unroll
            for (int i = 0; i < NFW; ++i) {
                const int f = wave + i * PN_WAVES;           // = tap * NKF + cf
                if (f < NKT) {
                    const int tap = f / NKF, cf = f - tap * NKF;
                    uint4 b = *reinterpret_cast<const uint4*>(&s_x[(c * 16 + jl + tap) * LD + (cf * KB + g * EPL) * (int)sizeof(XT)]);
                    if (!((tapmask[c] >> tap) & 1)) b = make_uint4(0, 0, 0, 0);
                    acc = mfma_frag<XT>(a[i], b, acc);
                }
            }
        }
        red[wave][c][lane] = acc;
    }
    __syncthreads();
    if (wave < PN_CT && ct0 + wave < n_ctiles) {
        floatx4 y = bias4;
#pragma unroll
        for (int w = 0; w < PN_WAVES; ++w) y += red[w][wave][lane];
        const int col = (ct0 + wave) * 16 + jl;
        const int ch = rt * 16 + 4 * g;                  // the lane holds channels ch .. ch + 3 of its column
        if constexpr (EPI != PN_EPI_LAST) {
            const float y0 = pn_act<EPI>(y[0]), y1 = pn_act<EPI>(y[1]), y2 = pn_act<EPI>(y[2]), y3 = pn_act<EPI>(y[3]);
            XT* dst = Xout + xoff<XT>(COUT / KB, col, ch);
            if constexpr (sizeof(XT) == 2) *reinterpret_cast<uint2*>(dst) = make_uint2(pack2<XT>(y0, y1), pack2<XT>(y2, y3));
            else *reinterpret_cast<float4*>(dst) = make_float4(y0, y1, y2, y3);
        } else {
            const int r = orow[col];
            if (r >= 0 && ch < n_mel) {
                const float4 m = *reinterpret_cast<const float4*>(mel + (size_t)col * n_mel + ch);
                *reinterpret_cast<float4*>(out + (size_t)r * n_mel + ch) = make_float4(m.x + y[0], m.y + y[1], m.z + y[2], m.w + y[3]);
            }
        }
    }
    if (EPI == PN_EPI_LAST && tid == 0) stamps.end();
}

// The same layer for large batches, and (TAPS = 1) the encoder's input projection: a workgroup owns WR x RPW row tiles and WC x CTW
// column tiles, RPW x CTW of them per wave.  K is not split, so nothing is reduced.  The columns are staged a few channel
// fragments at a time, the next ones on their way while the present ones are in use, all taps of a chunk before the next chunk.
//   * What a compute unit can take decides the shape.  Per k step (64 bytes of k) a wave fetches RPW KB of weights (16 cycles of
//     the unit's L1 a KB), reads CTW KB of operands from LDS (4.4 cycles a KB where nothing conflicts) and spends 17 RPW CTW
//     cycles in products: 2 x 2 waves of 2 x 4 tiles each take 128, 70 and 136 cycles of the unit.
//   * LDS holds a plane per 16 bytes of channels, rows = columns, planes a multiple of 16 pieces apart: the lanes of a B fragment
//     (16 columns x 4 pieces) then meet every bank once.  Operands are requested two steps ahead.
//   * A tap that leaves its window reads a row of zeros: an address chosen once per tap, not a mask on every operand (a vector
//     instruction beside a product costs it two to four cycles).  Which of the two buffers is read is a constant in the read's offset.
// The sums are those of the kernel above, bit for bit: eight partial sums, sum w of the fragments f = w, w + 8, ... (f = tap * NKF +
// channel fragment), added to the bias in the order of w.  So a request's and a chunk's results are the same alone and in a call of any
// size, whichever kernel a layer of the call takes.  A chunk holds the channel fragments w, w + 8, .. of one partial sum (fp32) or two
// (two-byte), or, with a few channels, all there are.  The price is 32 additions a wave and partial sum: with one chain over all of k,
// which differed from the kernel above by 1.4e-4 (two-byte) and was further off 64 bits in fp32 (1.5e-6 .. 1.7e-6 of the PostNet's output
// against 0.9e-6), a PostNet round of 64 / 256 requests took 68.7 / 163 us, like this 70.0 / 166 us; fp32 316 / 1047 us, like this 307 / 1032.
template <typename XT> constexpr int cc_ahead() { return sizeof(XT) == 2 ? 2 : 1; }   // k steps between an operand's request and its use
template <typename XT, int CIN, int TAPS, int CT, int WAVES> struct ColGeom {
    static constexpr int NKF = CIN / Frag<XT>::KB, NKT = TAPS * NKF;
    static constexpr bool PARTS = TAPS > 1;                    // (the input projection is one chain in its other kernel, too)
    static constexpr bool CHUNKED = NKF % PN_WAVES == 0;
    static constexpr int CF = CHUNKED ? 4 : NKF;               // channel fragments per chunk
    static constexpr int NCH = NKF / CF, BUFS = NCH > 1 ? 2 : 1;
    static constexpr int NK = TAPS * CF;                       // k steps per chunk
    static constexpr int CSTEP = PARTS && CHUNKED ? PN_WAVES / NCH : CF;   // between the first fragments of two chunks
    static constexpr int THREADS = WAVES * 64;
    static constexpr int HALO = TAPS / 2;
    static constexpr int ROWS = CT * 16 + 2 * HALO;            // staged columns; row ROWS is zero
    static constexpr int PLANE = (ROWS + 1 + 15) / 16 * 16;
    static constexpr int BUF_VECS = CF * 4 * PLANE;
    static constexpr int PIECES = CF * 4 * ROWS;
    static constexpr int PER = (PIECES + THREADS - 1) / THREADS;
    static constexpr int LDS = BUFS * BUF_VECS * 16;
    static constexpr int AHEAD = CHUNKED && PARTS && CT == 8 ? 4 : NK % 5 == 0 ? 5 : NK;    // weight fragments in flight (divides NK: the ring is static)
    static_assert(NKF % CF == 0 && NCH % BUFS == 0 && NK % AHEAD == 0, "whole chunks");
    // channel fragment (of the first chunk) that lies in place j of a chunk
    __device__ static constexpr int frag(int j) { return PARTS && NCH > 1 ? j * PN_WAVES / NKF + j % (NKF / PN_WAVES) * PN_WAVES : j; }
    // k step i of a chunk: the partial sum it belongs to (of the chunk's), how far in, its tap and its place in the chunk.  Where all
    // channels are one chunk, the first LONG partial sums have one fragment more than the others
    static constexpr int LONG = NKT % PN_WAVES, LEN = NKT / PN_WAVES, SPLIT = LONG * (LEN + 1);
    __device__ static constexpr int part(int i) { return !PARTS ? 0 : i < SPLIT ? i / (LEN + 1) : LONG + (i - SPLIT) / LEN; }
    __device__ static constexpr int within(int i) { return !PARTS ? i : i < SPLIT ? i % (LEN + 1) : (i - SPLIT) % LEN; }
    __device__ static constexpr int fragment(int i) { return PARTS ? part(i) + PN_WAVES * within(i) : i; }
    __device__ static constexpr int tap(int i) { return fragment(i) / NKF; }
    __device__ static constexpr int place(int i) { return !PARTS || NCH == 1 ? fragment(i) % NKF : part(i) * (NKF / PN_WAVES) + within(i) % (NKF / PN_WAVES); }
    static_assert(!PARTS || NCH == 1 || (LONG == 0 && NK % LEN == 0), "partial sums end with their chunk");
};

enum { CC_TANH = PN_EPI_TANH, CC_LAST = PN_EPI_LAST, CC_RELU = PN_EPI_RELU, CC_XPROJ = 3 };

struct ColArgs {
    const uint4* W;           // A-fragment order, k = tap * CIN + channel
    const uint4* W1;          // CC_XPROJ: the second half of the rows
    const float* bias;
    const float* bias1;
    const uint4* Xin;
    void* Xout;
    const int* cmeta;
    int n_ctiles;
    const float* mel;         // CC_LAST
    int n_mel;
    const int* orow;
    float* out;               // CC_LAST: [rows][n_mel]; CC_XPROJ: [2][max_cols][COUT / 2]
    int n_col, max_cols;      // CC_XPROJ
    Stamps stamps;            // CC_LAST: the call ends here
};

// grid = (row groups, ceil(column tiles / CT))
template <typename XT, int CIN, int COUT, int TAPS, int EPI, int WR, int WC, int RPW, int CTW>
__global__ __launch_bounds__(WR * WC * 64, 2) void k_conv_cols(ColArgs p)
{
    constexpr int CT = WC * CTW;
    using R = ColGeom<XT, CIN, TAPS, CT, WR * WC>;
    constexpr int NKF = R::NKF, CF = R::CF, NK = R::NK, AHEAD = R::AHEAD;
    constexpr bool PARTS = R::PARTS;
    extern __shared__ uint4 s_cols[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int rt_all = (blockIdx.x * WR + wave % WR) * RPW, cw = wave / WR * CTW;      // the wave's first row and column tile
    const bool half = EPI == CC_XPROJ && rt_all >= COUT / 32;
    const int rt0 = half ? rt_all - COUT / 32 : rt_all;
    const int ct0 = blockIdx.y * CT, n_col_pad = p.n_ctiles * 16, col_first = ct0 * 16 - R::HALO;

    // a fragment's place is a scalar offset: all weight loads share one address register
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(half ? p.W1 : p.W), 0, COUT / (EPI == CC_XPROJ ? 32 : 16) * R::NKT * 1024, BUFFER_RSRC_RAW);
    auto weight = [&](int chunk, int i, int r) __attribute__((always_inline)) {       // k step i of a chunk
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16, ((rt0 + r) * R::NKT + R::tap(i) * NKF + R::frag(R::place(i)) + chunk * R::CSTEP) * 1024, 0);
        return make_uint4(v.x, v.y, v.z, v.w);
    };
    // This thread's pieces of a chunk: piece = (plane, column).  The activations are read through a descriptor that begins at the tile
    // in front of the workgroup's (byte offsets stay small); a column outside them has an offset past its end, and reads zeros.
    const int tile0 = max(ct0 - 1, 0);
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(p.Xin + xfrag(NKF, tile0, 0, 0)), 0,
                                                                       min(p.n_ctiles - tile0, CT + 2) * NKF * 1024, BUFFER_RSRC_RAW);
    unsigned from[R::PER];
#pragma unroll
    for (int i = 0; i < R::PER; ++i) {
        const int idx = min(i * R::THREADS + tid, R::PIECES - 1), plane = idx / R::ROWS, col = col_first + idx - plane * R::ROWS;
        const bool in = col >= 0 && col < n_col_pad;
        from[i] = in ? (unsigned)xfrag(NKF, (col >> 4) - tile0, R::frag(plane >> 2), (col & 15) + 16 * (plane & 3)) * 16u : 0x80000000u;
    }
    uint4 st[R::PER];
    auto request = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < R::PER; ++i) {
            const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)from[i], chunk * R::CSTEP * 1024, 0);
            st[i] = make_uint4(v.x, v.y, v.z, v.w);
        }
    };
    auto stash = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < R::PER; ++i) {
            const int idx = i * R::THREADS + tid, plane = idx / R::ROWS;
            if ((i + 1) * R::THREADS <= R::PIECES || idx < R::PIECES) s_cols[buf * R::BUF_VECS + plane * R::PLANE + idx - plane * R::ROWS] = st[i];
        }
    };
    request(0);
    uint4 ring[AHEAD][RPW];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
#pragma unroll
        for (int r = 0; r < RPW; ++r) ring[i][r] = weight(0, i, r);
    for (int i = tid; i < R::BUFS * CF * 4; i += R::THREADS) s_cols[i * R::PLANE + R::ROWS] = make_uint4(0, 0, 0, 0);
    // where every tap's operand lies: the column it meets, or a row of zeros where it leaves the column's own window
    const uint4* at[TAPS][CTW];
#pragma unroll
    for (int c = 0; c < CTW; ++c) {
        const int m = TAPS > 1 ? p.cmeta[min((ct0 + cw + c) * 16 + n, n_col_pad - 1)] : 0;
        const int t = m & 0xFFFF, T = m >> 16;
#pragma unroll
        for (int tap = 0; tap < TAPS; ++tap)
            at[tap][c] = s_cols + g * R::PLANE + (TAPS == 1 || (unsigned)(t + tap - R::HALO) < (unsigned)T ? (cw + c) * 16 + n + tap : R::ROWS);
    }
    floatx4 acc[RPW][CTW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const floatx4 b = *reinterpret_cast<const floatx4*>((half ? p.bias1 : p.bias) + (rt0 + r) * 16 + 4 * g);
#pragma unroll
        for (int c = 0; c < CTW; ++c) acc[r][c] = b;
    }
    // A partial sum is added when its successor begins, tile by tile between the products: behind its own last product every addition would
    // wait for the matrix pipe.  (Pinned there: left to itself the compiler adds all of them at the end, and keeps them in scratch memory.)
    floatx4 part[PARTS ? RPW : 1][PARTS ? CTW : 1];
    if constexpr (PARTS) {
#pragma unroll
        for (int r = 0; r < RPW; ++r)
#pragma unroll
            for (int c = 0; c < CTW; ++c) part[r][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    auto add_part = [&](int r, int c) __attribute__((always_inline)) {
        acc[r][c] += part[r][c];
        asm volatile("" : "+v"(acc[r][c]));
    };
    stash(0);
    __syncthreads();
    constexpr int CC_AHEAD = cc_ahead<XT>(), NB = CC_AHEAD + 1;
    auto do_chunk = [&](int chunk, int buf) __attribute__((always_inline)) {      // buf: a constant, so that it is part of a read's offset
        const int next = min(chunk + 1, R::NCH - 1);           // the last chunk requests its own first weights again, and drops them
        if (chunk + 1 < R::NCH) request(chunk + 1);
        uint4 bv[NB][CTW];
        auto operands = [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < CTW; ++c) bv[i % NB][c] = at[R::tap(i)][c][buf * R::BUF_VECS + R::place(i) * 4 * R::PLANE];
        };
#pragma unroll
        for (int i = 0; i < CC_AHEAD; ++i) operands(i);
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            uint4 af[RPW];
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                af[r] = ring[i % AHEAD][r];
                if (i + AHEAD < NK) ring[i % AHEAD][r] = weight(chunk, i + AHEAD, r);
                else if constexpr (R::NCH > 1) ring[i % AHEAD][r] = weight(next, i + AHEAD - NK, r);
            }
            if (i + CC_AHEAD < NK) operands(i + CC_AHEAD);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < CTW; ++c)
#pragma unroll
                for (int r = 0; r < RPW; ++r) {
                    if constexpr (PARTS) {
                        if (R::within(i) == 0) add_part(r, c);
                        part[r][c] = mfma_frag<XT>(af[r], bv[i % NB][c], R::within(i) == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : part[r][c]);
                    } else acc[r][c] = mfma_frag<XT>(af[r], bv[i % NB][c], acc[r][c]);
                }
        }
        if (chunk + 1 < R::NCH) {
            stash(buf ^ 1);
            lds_barrier();
        }
    };
#pragma unroll 1
    for (int chunk = 0; chunk < R::NCH; chunk += R::BUFS) {
        do_chunk(chunk, 0);
        if constexpr (R::BUFS == 2) do_chunk(chunk + 1, 1);
    }
#pragma unroll
    for (int c = 0; c < CTW; ++c) {
        if (ct0 + cw + c >= p.n_ctiles) break;
        if constexpr (PARTS) {
#pragma unroll
            for (int r = 0; r < RPW; ++r) acc[r][c] += part[r][c];
        }
        const int col = (ct0 + cw + c) * 16 + n;
        const int r_out = EPI == CC_LAST ? p.orow[col] : 0;
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            const floatx4 y = acc[r][c];
            const int ch = (rt0 + r) * 16 + 4 * g;
            if constexpr (EPI == CC_XPROJ) {
                if (col < p.n_col) *reinterpret_cast<floatx4*>(p.out + ((size_t)(half ? 1 : 0) * p.max_cols + col) * (COUT / 2) + ch) = y;
            } else if constexpr (EPI == CC_LAST) {
                if (r_out >= 0 && ch < p.n_mel) {
                    const float4 m = *reinterpret_cast<const float4*>(p.mel + (size_t)col * p.n_mel + ch);
                    *reinterpret_cast<float4*>(p.out + (size_t)r_out * p.n_mel + ch) = make_float4(m.x + y[0], m.y + y[1], m.z + y[2], m.w + y[3]);
                }
            } else {
                const float y0 = pn_act<EPI>(y[0]), y1 = pn_act<EPI>(y[1]), y2 = pn_act<EPI>(y[2]), y3 = pn_act<EPI>(y[3]);
                XT* dst = reinterpret_cast<XT*>(p.Xout) + xoff<XT>(COUT / Frag<XT>::KB, col, ch);
                if constexpr (sizeof(XT) == 2) *reinterpret_cast<uint2*>(dst) = make_uint2(pack2<XT>(y0, y1), pack2<XT>(y2, y3));
                else *reinterpret_cast<float4*>(dst) = make_float4(y0, y1, y2, y3);
            }
        }
    }
    if (EPI == CC_LAST && tid == 0) p.stamps.end();
}

// 2 x 2 waves of two row tiles each; five waves of one where there are five (the PostNet's last layer); four waves of two row
// tiles each in the input projection, which has few k steps and whose time is its stores (16 requests of 165 tokens 26.8 -> 16.2 us;
// 2 x 2 waves 16.8, and 50.6 against 42.7 us for 64 requests)
template <int COUT, int TAPS> struct ColWaves {
    static constexpr bool FOUR = COUT / 16 % 4 == 0, SQUARE = FOUR && TAPS > 1;
    static constexpr int WR = SQUARE ? 2 : FOUR ? 4 : COUT / 16, WC = SQUARE ? 2 : 1, RPW = FOUR ? 2 : 1, GROUPS = COUT / 16 / (WR * RPW);
    static constexpr int CT_MOST = SQUARE ? 8 : FOUR ? 7 : 4;
};

template <typename XT, int CIN, int COUT, int TAPS, int EPI, int CT>
inline hipError_t conv_cols_ct(const ColArgs& p, hipStream_t s)
{
    using V = ColWaves<COUT, TAPS>;
    using R = ColGeom<XT, CIN, TAPS, CT, V::WR * V::WC>;
    static_assert(V::GROUPS * V::WR * V::RPW * 16 == COUT && V::WR * V::WC <= 8 && CT % V::WC == 0, "whole row and column groups");
    auto kern = k_conv_cols<XT, CIN, COUT, TAPS, EPI, V::WR, V::WC, V::RPW, CT / V::WC>;
    static bool attr_set = false;                 // dynamic LDS above 64 KB has to be allowed once per kernel
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, R::LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(V::GROUPS, (p.n_ctiles + CT - 1) / CT), dim3(R::THREADS), R::LDS, s, p);
    return hipGetLastError();
}

// Column tiles of a call from which a layer takes the kernel above (the sums are the same, so every layer has a line of its own).
// (Small calls of the PostNet and the encoder are one launch, conv5_chain.h; the lines below those sizes are for tts_postnet_run_static.)
// Launches in us, small-call kernel / the kernel above:
//   two-byte  512 -> 512     20 tiles  8.4 /  8.2,   24  8.8 /  8.4,   36 10.8 /  8.7,   79 16.9 / 10.3
//             96 -> 512      20        4.2 /  3.8,   36  4.8 /  4.1,   79  6.9 /  5.3
//             projection     20        5.5 /  5.1,   24  5.2 /  5.5,   28  7.4 /  5.9,   79 13.6 / 10.0
//             512 -> 80      79        5.3 /  7.4,  100  6.0 /  8.1,  128  8.1 /  8.0,  256 12.3 /  7.9
//   fp32      512 -> 512     24       22.0 / 23.1,   28 27.7 / 23.3,   40 35.2 / 23.7,   79 65.0 / 41.8
//             96 -> 512      24        6.2 /  7.8,   28  7.3 /  7.6,   36  9.6 /  8.2,   79 13.0 / 12.9
//             projection     36       17.0 / 19.9,   79 31.4 / 34.3,  128 48.5 / 60.3,  160 60.2 / 61.2,  200 74.0 / 62.2
//             512 -> 80      79       16.2 / 38.4,  200 30.2 / 38.5,  256 36.4 / 38.4,  320 48.4 / 38.8
// (512 -> 80 has five row tiles only: above, a workgroup has all of K in a chain, whatever the size of the call.  The projection in fp32
// changes sides three times between 28 and 160 tiles with the last wave of its workgroups, by 3 us up to 100 tiles.)
// (512 -> 512 and 96 -> 512, two-byte: traced launch by launch, as above, the kernels meet at 20 tiles; queued one behind the other the
// small-call kernel's layer of 512 channels is the faster one up to 32, where its 32 x n / 2 workgroups are two for every compute unit.  PostNet
// calls of 25 / 28 / 32 tiles with both lines at 25 45.4 / 46.0 / 46.5 us, at 33 45.0 / 45.6 / 45.6, at 25 and 33 44.8 / 44.8 / 45.5; encoder
// calls 82.2 / 82.8 / 83.6 with 25, 80.4 / 81.3 / 82.5 with 33.  In fp32, one column tile a workgroup, the 25th tile begins a fourth workgroup.)
template <typename XT, int CIN, int COUT, int TAPS> constexpr int cols_from()
{
    constexpr bool TWO_BYTE = sizeof(XT) == 2;
    if constexpr (TAPS == 1) return TWO_BYTE ? 25 : 160;
    else if constexpr (COUT == PN_COUT_LAST) return TWO_BYTE ? 128 : 260;
    else return TWO_BYTE && CIN == 512 ? 33 : 25;
}

// Column tiles per workgroup: the fewest that leave no more workgroups than there are compute units, CT_MOST at most (up to there
// the registers hold the sums and two workgroups share a CU's LDS)
constexpr int CC_CUS = 256;
template <typename XT, int CIN, int COUT, int TAPS, int EPI>
inline hipError_t conv_cols(const ColArgs& p, hipStream_t s)
{
    using V = ColWaves<COUT, TAPS>;
    auto fits = [&](int ct) { return V::GROUPS * ((p.n_ctiles + ct - 1) / ct) <= CC_CUS; };
    constexpr int LEAST = cols_from<XT, CIN, COUT, TAPS>();         // forms that no call of so many column tiles takes are not built
    if constexpr (V::GROUPS * ((LEAST + 1) / 2) <= CC_CUS)
        if (fits(2)) return conv_cols_ct<XT, CIN, COUT, TAPS, EPI, 2>(p, s);
    constexpr int MOST = sizeof(XT) == 4 && CIN < 512 ? 4 : V::CT_MOST;       // (fp32, few channels: 320 tiles 29 us in fours, 38 in eights; 800: 60, 69)
    if constexpr (MOST == 4 || V::GROUPS * ((LEAST + 3) / 4) <= CC_CUS)
        if (MOST == 4 || fits(4)) return conv_cols_ct<XT, CIN, COUT, TAPS, EPI, 4>(p, s);
    return conv_cols_ct<XT, CIN, COUT, TAPS, EPI, MOST>(p, s);
}

template <typename XT, int CIN, int COUT, int EPI>
inline hipError_t conv_layer(const void* W, const float* b, const void* xin, XT* xout, const int* cmeta, int n_ctiles,
                             const float* mel, int n_mel, const int* orow, float* out, const Stamps& stamps, hipStream_t s)
{
    if (n_ctiles >= cols_from<XT, CIN, COUT, PN_TAPS>()) {
        ColArgs p{};
        p.W = (const uint4*)W;
        p.bias = b;
        p.Xin = (const uint4*)xin;
        p.Xout = xout;
        p.cmeta = cmeta;
        p.n_ctiles = n_ctiles;
        p.mel = mel;
        p.n_mel = n_mel;
        p.orow = orow;
        p.out = out;
        p.stamps = stamps;
        return conv_cols<XT, CIN, COUT, PN_TAPS, EPI>(p, s);
    } else {
        constexpr int CT = PnCT<XT>::value;
        const dim3 grid(COUT / 16, (n_ctiles + CT - 1) / CT);
        hipLaunchKernelGGL((k_pn_conv<XT, CIN, COUT, EPI>), grid, dim3(PN_THREADS), 0, s, (const uint4*)W, b, (const uint4*)xin,
                           xout, cmeta, n_ctiles, mel, n_mel, orow, out, stamps);
    }
    return hipGetLastError();
}

}  // namespace tts
