// A segment of decoder steps as ONE launch for pools with fp32 weights and memory whose running requests lie in the first 16 slots: the
// counterpart of segment.hip, which says how such a launch works (words, their three buffers, the two sets, the bounded waits) and why it pays.
//
// As launches of its own (four, kernels.hip) a step takes 38.9 us at 16 requests of 60 positions and 37.3 at one: 15 of them one leader's prenet and
// the gate pre-sums behind it, 10 the attention, 14 the two LSTMs, each with its start-up, a cold trip and its share of 73 MB of weights.  Like this
// 16.9 and 14.9; 16 requests of 250 positions 39.9 -> 19.5.  Twice the bytes of the two-byte form and an eighth of its matrix rate (256 FLOP a cycle
// and compute unit; the products of a step are 10 us of 96 units) ask for another split of the work:
//   32 x ATT    32 hidden units of the attention LSTM each: gates from p (K = 256) and the pre-sums (words), cell, h, rank-32 share of the query
//  128 x GATES  8 hidden units of the decoder LSTM and of the attention LSTM's pre-sums each.  In a step: the decoder's sums over h_att (while the
//               attention works), over a (on the chain), cell, h_dec out; then, off the chain, the attention LSTM's pre-sums of the next step over
//               [a; h_att], and the decoder's over h_dec.  The decoder's weights live in registers and LDS (328 KB), the pre-sums' (196 KB)
//               stream from L2: 16 such workgroups an XCD, 3 MB of its 4.
//   S x LSA     per request; S = 4 up to 8 slots, 2 above; 448 and 224 positions of its memory stay in registers and LDS (with 256 and 128, in
//               registers alone, 16 requests of 165 / 250 positions 19.2 / 20.7 us a step, like this 18.8 / 19.5)
//    6 x ROWS   one row tile of the projection each
//    4 x LEAD   frame and the prenet's first layer each, a quarter of its second: a chain of 64 matrix instructions a row tile, four row tiles
//               side by side on the SIMDs (one workgroup for all of it: 3.4 us); the first one keeps the books
// The chain of a step at 16 requests of 60 positions, us from p's arrival: query stored 2.5 (1.7 of them products: 64 matrix instructions in a
// chain a row tile, two a SIMD), taken 3.6, energies stored 5.8, taken 6.3, context stored 7.0, taken 8.8, h_dec stored 10.3, taken 11.9, frame's sums stored
// 13.2, taken 14.2, prenet stored 16.7, taken 17.6.  (Pauses between the polls change nothing.)
// Every sum is formed in the order of the kernels in kernels.hip: the same bits whichever form a step takes.
#include "kernels.h"
#include "lsa_tile.h"
#include "mfma.h"
#include "segment_parts.h"
#include "words.h"

namespace tts {
namespace {

constexpr int KB = Frag<float>::KB;
constexpr int NK_A = K_ATT / KB, NK_D = K_DEC / KB, NK_P = K_PROJ / KB;    // fragments per row tile: 112, 160, 96
constexpr int F_H = HID / KB, F_A = ENC / KB, F_P = PRENET / KB;            // fragments of h, a, p: 64, 32, 16
static_assert(F_H == 8 * NW && F_A == 4 * NW && F_P == 2 * NW, "a wave takes eight fragments of h, four of a, two of p");
constexpr int MEL_ROWS = 96, GATES = 128;

// One buffer of each kind, in bytes; what one workgroup (for q and p: one wave) stores lies together
constexpr int B_FRAG = 1024, B_H = F_H * B_FRAG, B_A = F_A * B_FRAG, B_P = F_P * B_FRAG, B_PRE = HID / 4 * 1024;
constexpr int B_QS = QUERY_PARTIALS * ATT * 4, B_Q = SEG_SLOTS * B_QS, B_M = SEG_SLOTS * MEL_ROWS * 4;
constexpr int O_HA = 0, O_HD = O_HA + 3 * B_H, O_A = O_HD + 3 * B_H, O_P = O_A + 3 * B_A, O_PRE = O_P + 3 * B_P, O_Q = O_PRE + 3 * B_PRE, O_M = O_Q + 3 * B_Q,
              O_E = O_M + 3 * B_M;
static_assert(O_E == SEG32_FIXED_BYTES, "the arena's share");

// a lane's offset in a fragment: of h_att and p ([fragment][slot][16]), of h_dec ([half a fragment][slot][8]) and of a ([slot][512])
__device__ __forceinline__ int off_hp(int col, int g) { return col * 64 + g * 16; }
__device__ __forceinline__ int off_hd(int col, int g) { return ((g >> 1) * SEG_SLOTS + col) * 32 + (g & 1) * 16; }
__device__ __forceinline__ int off_a(int col, int g) { return col * (ENC * 4) + g * 16; }

// Words::take for fragments at at(0), at(1), ...
template <int N, int NAP, class AT>
__device__ __forceinline__ bool take_at(const Words& x, int lane_off, bool on, AT at, uint4 (&out)[N])
{
    u32x4_t w[N];
#pragma unroll
    for (int n = 0; n < N; ++n) w[n] = u32x4_t{0u, 0u, 0u, 0u};
    bool in = !on;
    for (int spin = 0; spin < x.polls && !in; ++spin) {
        Words::again();
#pragma unroll
        for (int n = 0; n < N; ++n) w[n] = x.look4(lane_off, at(n));
        in = true;
#pragma unroll
        for (int n = 0; n < N; ++n) in = in && Words::full(w[n]);
        if constexpr (NAP > 0) {
            if (!in) __builtin_amdgcn_s_sleep(NAP);
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n) out[n] = as_uint4(w[n]);
    return in;
}

constexpr int S_ATT = F_P * 1024 + 32 * 16 * 4;
constexpr int G_LDS = 6;                                    // of a wave's eight fragments of h_dec, those whose weights lie in LDS (per row tile)
constexpr int S_RED = NW * 2 * 1024, S_GATES = 3 * S_RED + NW * 2 * G_LDS * 1024;
constexpr int P_LD = 68;
constexpr int S_ROWS = 6 * NW * 4 * P_LD * 4;
constexpr int MEL_LD = MEL_ROWS + 4, HID_LD = PRENET + 4;     // an odd number of 16-byte pieces a row
constexpr int S_LEAD = 16 * (MEL_LD + HID_LD) * 4;
constexpr int U_PAD = MAX_ENC_LEN + 48;
constexpr int S_LSA = (NW * ENC + 16 * ATT + 2 * U_PAD + MAX_ENC_LEN + 2 * ATT + 2 * NW + 32 * 64 + 8 * 64 * 4) * 4;
// Beside what it needs LDS holds the rows of so many positions of a request's memory that the workgroup's columns of them are 96 KB.
constexpr int S_ROWS_KEPT = 96 * 1024, S_MAX = S_LSA + S_ROWS_KEPT;
constexpr int lsa_lds_passes(int split) { return S_ROWS_KEPT / (32 * ENC * 4 / split); }
static_assert(lsa_lds_passes(2) == 3 && lsa_lds_passes(4) == 6, "224 and 448 positions with those in registers");
static_assert(S_ATT <= S_MAX && S_GATES <= S_MAX && S_ROWS <= S_MAX && S_LEAD <= S_MAX && S_LSA % 16 == 0 && S_MAX + 128 <= 160 * 1024, "the roles' LDS");

// ---------------------------------------------------------------- the attention LSTM and the query
__device__ __forceinline__ void att(const DevPtrs& d, const Words& x, const Pool& pl, int rg, char* lds, Phases ps)
{
    const int wave = wave_id(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4, cur = pl.cur;
    const int rt = rg * 8 + wave, unit = rt * 4 + g, rem = pl.rem[col];
    uint4 (*s_b)[64] = reinterpret_cast<uint4 (*)[64]>(lds);
    float (*s_h)[16] = reinterpret_cast<float (*)[16]>(lds + F_P * 1024);
    uint4 we[F_P];
#pragma unroll
    for (int f = 0; f < F_P; ++f) we[f] = d.Wa[xfrag(NK_A, rt, f, lane)];
    float wq[8];                                            // W_q[16 wave + ..][32 rg + 4 k + ..]
#pragma unroll
    for (int k = 0; k < 8; ++k) wq[k] = d.Wq_epi[((size_t)(rg * 8 + k) * 8 + wave) * 64 + lane];
    const floatx4 bias4 = *reinterpret_cast<const floatx4*>(d.ba + unit * 4);
    float* c_g = d.c_att + (size_t)col * HID + unit;
    floatx4 pre4 = reinterpret_cast<const floatx4*>(d.pre_att)[(size_t)rt * 64 + lane];
    float c = c_g[0];
    const int q_off = col * B_QS + (16 * wave + 4 * g) * 4;
    int b = 0, b_before = 2, b_next = 1;
    for (int s = 0; s < pl.n_steps; ++s) {
        const bool on = s < rem;
        bool ok = true;
        uint4 pb[2];
        if (s > 0) {
            uint4 pre[1];
            ok = take_at<1, 4>(x, lane * 16, on, [&](int) { return O_PRE + b_before * B_PRE + rt * B_FRAG; }, pre);
            pre4 = __builtin_bit_cast(floatx4, pre[0]);
            ok = take_at<2, 0>(x, off_hp(col, g), on, [&](int n) { return O_P + b_before * B_P + (wave + 8 * n) * B_FRAG; }, pb) && ok;
        } else {
#pragma unroll
            for (int n = 0; n < 2; ++n) pb[n] = reinterpret_cast<const uint4*>(d.xatt[cur])[xfrag(NK_A, 0, wave + 8 * n, lane)];
        }
        stores_done();
        s_b[wave][lane] = pb[0];
        s_b[wave + 8][lane] = pb[1];
        ps.sync(ok);
        floatx4 g4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < F_P; ++f) g4 = mfma_frag<float>(we[f], s_b[f][lane], g4);
        g4 += bias4;
        g4 += pre4;
        float c_new = c, h;
        cell(g4, c_new, h);
        s_h[4 * wave + g][col] = on ? h : 0.f;
        if (ps.bad()) return give_up(d, pl, s);
        lds_barrier();
        // the units' share of the query: 16 rows per wave
        {
            floatx4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 8; ++k) part = __builtin_amdgcn_mfma_f32_16x16x4f32(wq[k], s_h[4 * k + g][col], part, 0, 0, 0);
            if (on) x.put4(part, q_off, O_Q + b * B_Q + rg * ATT * 4);
            if (wave < 2 && on) {
                floatx4 hv;
#pragma unroll
                for (int i = 0; i < 4; ++i) hv[i] = s_h[16 * wave + 4 * g + i][col];
                x.put4(hv, off_hp(col, g), O_HA + b * B_H + (2 * rg + wave) * B_FRAG);
            }
        }
        if (on) c = c_new;
        if (s + 1 == min(rem, pl.n_steps)) {
            // the request's last step of this segment: its state where the step kernels keep it
            const int end = cur ^ ((s + 1) & 1);
            c_g[0] = c;
            reinterpret_cast<float*>(d.xatt[end])[xoff<float>(NK_A, col, XA_H + unit)] = h;
            reinterpret_cast<float*>(d.xdec[end ^ 1])[xoff<float>(NK_D, col, XD_HA + unit)] = h;
        }
        // Step s - 1's words, whose buffer is step s + 2's: their readers were done before this step's p could be made (its frame's sums need
        // all of h_dec, and that every h_att and every a, made of every q)
        if (on) x.empty4(q_off, O_Q + b_before * B_Q + rg * ATT * 4);
        if (wave < 2 && on) x.empty4(off_hp(col, g), O_HA + b_before * B_H + (2 * rg + wave) * B_FRAG);
        b_before = b;
        b = b_next;
        b_next = next3(b);
    }
}

// ---------------------------------------------------------------- the decoder LSTM, and the attention LSTM's pre-sums
__device__ __forceinline__ void gates(const DevPtrs& d, const Words& x, const Pool& pl, int j, char* lds, Phases ps)
{
    const int wave = wave_id(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4, cur = pl.cur, n_steps = pl.n_steps;
    // three reduction buffers, one after the other in a step: what was read from one is done when the barrier of the next has been passed
    floatx4 (*red0)[2][64] = reinterpret_cast<floatx4 (*)[2][64]>(lds);
    floatx4 (*red1)[2][64] = red0 + NW;
    floatx4 (*red2)[2][64] = red1 + NW;
    uint4* s_w = reinterpret_cast<uint4*>(lds + 3 * S_RED) + wave * 2 * G_LDS * 64 + lane;       // the wave's own
    uint4 w_ha[2][8], w_a[2][4], w_hd[2][8 - G_LDS];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
#pragma unroll
        for (int f = 0; f < 8; ++f) w_ha[r][f] = d.Wd[xfrag(NK_D, 2 * j + r, wave + 8 * f, lane)];
#pragma unroll
        for (int f = 0; f < 4; ++f) w_a[r][f] = d.Wd[xfrag(NK_D, 2 * j + r, wave + 8 * (8 + f), lane)];
#pragma unroll
        for (int f = 0; f < 8 - G_LDS; ++f) w_hd[r][f] = d.Wd[xfrag(NK_D, 2 * j + r, wave + 8 * (12 + f), lane)];
#pragma unroll
        for (int f = 0; f < G_LDS; ++f) s_w[(r * G_LDS + f) * 64] = d.Wd[xfrag(NK_D, 2 * j + r, wave + 8 * (20 - G_LDS + f), lane)];
    }
    // the pre-sums' weights: a fragment's place is a scalar offset, all loads share one address register
    const __amdgpu_buffer_rsrc_t wa = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(d.Wa + xfrag(NK_A, 2 * j, 0, 0)), 0, 2 * NK_A * 1024, BUFFER_RSRC_RAW);
    auto late = [&](int r, int f) __attribute__((always_inline)) {
        return __builtin_amdgcn_raw_buffer_load_b128(wa, lane * 16, (r * NK_A + wave + 8 * (2 + f)) * 1024, 0);
    };
    const int er = wave & 1, rt = 2 * j + er, unit = rt * 4 + g, rem = pl.rem[col];
    const int hd_off = col * 32 + er * 16 + g * 4, hd_at = O_HD + j * (B_FRAG / 2), pre_at = O_PRE + rt * B_FRAG;
    const floatx4 bias4 = *reinterpret_cast<const floatx4*>(d.bd + unit * 4);
    float* c_g = d.c_dec + (size_t)col * HID + unit;
    floatx4 pre4 = reinterpret_cast<const floatx4*>(d.pre_dec)[(size_t)rt * 64 + lane];
    float c = c_g[0];
    auto sum = [&](floatx4 (*red)[2][64]) __attribute__((always_inline)) {
        floatx4 v = red[0][er][lane];
#pragma unroll
        for (int k = 1; k < NW; ++k) v += red[k][er][lane];
        return v;
    };
    constexpr int AHEAD = 3;
    int b = 0, b_next = 1;
    for (int s = 0; s < n_steps; ++s) {
        const bool on = s < rem, mine = wave < 2 && on;
        // ahead of the chain: the decoder's sums over h_att
        uint4 ha[8], ab[4];
        bool ok = take_at<8, 4>(x, off_hp(col, g), on, [&](int n) { return O_HA + b * B_H + (wave + 8 * n) * B_FRAG; }, ha);
        // (step s - 2's words: read before this h_att could be made)
        if (mine) {
            x.empty(hd_off, hd_at + b_next * B_H);
            x.empty4(lane * 16, pre_at + b_next * B_PRE);
        }
        floatx4 acc[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < 8; ++f)
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[r] = mfma_frag<float>(w_ha[r][f], ha[f], acc[r]);
        ok = take_at<4, 0>(x, off_a(col, g), on, [&](int n) { return O_A + b * B_A + (wave + 8 * n) * 64; }, ab) && ok;
        stores_done();
        u32x4_t ring[AHEAD][2];
#pragma unroll
        for (int f = 0; f < AHEAD; ++f)
#pragma unroll
            for (int r = 0; r < 2; ++r) ring[f][r] = late(r, f);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[r] = mfma_frag<float>(w_a[r][f], ab[f], acc[r]);
#pragma unroll
        for (int r = 0; r < 2; ++r) red0[wave][r][lane] = acc[r];
        ps.sync(ok);
        {
            floatx4 g4 = bias4;
#pragma unroll
            for (int k = 0; k < NW; ++k) g4 += red0[k][er][lane];
            g4 += pre4;
            float c_new = c, h;
            cell(g4, c_new, h);
            if (ps.bad()) return give_up(d, pl, s);
            // (waves 2 .. 7 form the same cells and store nothing)
            if (mine) x.put(__float_as_uint(h), hd_off, hd_at + b * B_H);
            if (on) c = c_new;
            if (wave < 2 && s + 1 == min(rem, n_steps)) {
                c_g[0] = c;
                reinterpret_cast<float*>(d.xdec[cur ^ ((s + 1) & 1)])[xoff<float>(NK_D, col, XD_HD + unit)] = h;
            }
        }
        // off the chain: the attention LSTM's pre-sums over [a; h_att] for the next step
#pragma unroll
        for (int r = 0; r < 2; ++r) acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < 12; ++f) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const uint4 w = as_uint4(ring[f % AHEAD][r]);
                if (f + AHEAD < 12) ring[f % AHEAD][r] = late(r, f + AHEAD);
                acc[r] = mfma_frag<float>(w, f < 4 ? ab[f < 4 ? f : 0] : ha[f < 4 ? 0 : f - 4], acc[r]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) red1[wave][r][lane] = acc[r];
        lds_barrier();
        {
            const floatx4 v = sum(red1);
            if (mine) {
                if (s + 1 < n_steps) x.put4(v, lane * 16, pre_at + b * B_PRE);
                else reinterpret_cast<floatx4*>(d.pre_att)[(size_t)rt * 64 + lane] = v;
            }
        }
        // and the decoder's over this step's h_dec
        {
            uint4 hd[8];
            ok = take_at<8, 2>(x, off_hd(col, g), on, [&](int n) { return O_HD + b * B_H + (wave + 8 * n) * B_FRAG; }, hd);
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int f = 0; f < 8; ++f)
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    acc[r] = mfma_frag<float>(f < 8 - G_LDS ? w_hd[r][f < 8 - G_LDS ? f : 0] : s_w[(r * G_LDS + f - (8 - G_LDS)) * 64], hd[f], acc[r]);
#pragma unroll
            for (int r = 0; r < 2; ++r) red2[wave][r][lane] = acc[r];
            ps.sync(ok);
            pre4 = sum(red2);
            if (ps.bad()) return give_up(d, pl, s);
            if (mine && s + 1 == n_steps) reinterpret_cast<floatx4*>(d.pre_dec)[(size_t)rt * 64 + lane] = pre4;
        }
        b = b_next;
        b_next = next3(b);
    }
}

// ---------------------------------------------------------------- one row tile of the projection
__device__ __forceinline__ void rows(const DevPtrs& d, const Words& x, const Pool& pl, int r, char* lds, Phases ps)
{
    const int wave = wave_id(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    float (*part)[NW][4][P_LD] = reinterpret_cast<float (*)[NW][4][P_LD]>(lds);  // [sixth of K][wave][element of the accumulator][lane]
    // a wave's two fragments of sixth kp: 16 kp + 2 wave, + 1
    uint4 w[6][2];
#pragma unroll
    for (int kp = 0; kp < 6; ++kp)
#pragma unroll
        for (int i = 0; i < 2; ++i) w[kp][i] = reinterpret_cast<const uint4*>(d.Wmel)[((size_t)r * NK_P + 16 * kp + 2 * wave + i) * 64 + lane];
    const int rem = pl.rem[col];
    // in the reduction: wave = four columns, thread = one of them and one of 16 rows
    const int my_col = (4 * wave + g) & 15, row16 = lane & 15, row = 16 * r + row16;
    const int el = row16 & 3, at = my_col + 16 * (row16 >> 2), m_off = (my_col * 16 + row16) * 4, m_buf = O_M + r * (SEG_SLOTS * 64);
    const int my_rem = wave < 4 && row < N_PROJ ? pl.rem[my_col] : 0;
    const float bias = d.bmel[min(row, N_PROJ - 1)];
    auto product = [&](int kp, const uint4& b0, const uint4& b1) __attribute__((always_inline)) {
        floatx4 p = mfma_frag<float>(w[kp][0], b0, floatx4{0.f, 0.f, 0.f, 0.f});
        p = mfma_frag<float>(w[kp][1], b1, p);
#pragma unroll
        for (int i = 0; i < 4; ++i) part[kp][wave][i][lane] = p[i];
    };
    auto sixth = [&](int kp) __attribute__((always_inline)) {
        float v = kp == 0 ? bias : 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) v += part[kp][k][el][at];
        return v;
    };
    int b = 0, b_next = 1;
    for (int s = 0; s < pl.n_steps; ++s) {
        const bool on = s < rem;
        uint4 ab[4], hd[8];
        bool ok = take_at<4, 8>(x, off_a(col, g), on, [&](int n) { return O_A + b * B_A + (16 * (n >> 1) + 2 * wave + (n & 1)) * 64; }, ab);
        if (s < my_rem) x.empty(m_off, m_buf + b_next * B_M);
        product(4, ab[0], ab[1]);
        product(5, ab[2], ab[3]);
        ps.sync(ok);
        const float v4 = sixth(4), v5 = sixth(5);
        if (ps.bad()) return give_up(d, pl, s);
        ok = take_at<8, 0>(x, off_hd(col, g), on, [&](int n) { return O_HD + b * B_H + (16 * (n >> 1) + 2 * wave + (n & 1)) * B_FRAG; }, hd);
        stores_done();
#pragma unroll
        for (int kp = 0; kp < 4; ++kp) product(kp, hd[2 * kp], hd[2 * kp + 1]);
        ps.sync(ok);
        float v = sixth(0);
#pragma unroll
        for (int kp = 1; kp < 4; ++kp) v += sixth(kp);
        v += v4;
        v += v5;
        if (ps.bad()) return give_up(d, pl, s);
        if (s < my_rem) x.put(__float_as_uint(v), m_off, m_buf + b * B_M);
        b = b_next;
        b_next = next3(b);
    }
}

// ---------------------------------------------------------------- frame, prenet, books
__device__ __forceinline__ void lead(const DevPtrs& d, const Words& x, const Pool& pl, int quarter, char* lds, Phases ps)
{
    const int tid = threadIdx.x, wave = wave_id(), lane = tid & 63, col = lane & 15, g = lane >> 4;
    const int cur = pl.cur, n_steps = pl.n_steps;
    float (*s_mel)[MEL_LD] = reinterpret_cast<float (*)[MEL_LD]>(lds);
    float (*s_hid)[HID_LD] = reinterpret_cast<float (*)[HID_LD]>(lds + 16 * MEL_LD * 4);
    constexpr int NK3 = N_MEL / KB, NK4 = PRENET / KB;
    uint4 a3[2][NK3], a4[NK4];
    const int mt = 4 * quarter + (wave & 3);                 // waves 0 .. 3: a row tile of the second layer
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int f = 0; f < NK3; ++f) a3[m][f] = reinterpret_cast<const uint4*>(d.Wp1)[((size_t)(wave + 8 * m) * NK3 + f) * 64 + lane];
#pragma unroll
    for (int f = 0; f < NK4; ++f) a4[f] = reinterpret_cast<const uint4*>(d.Wp2)[((size_t)mt * NK4 + f) * 64 + lane];
    const int rem = pl.rem[col];
    // as a collector of the frame: thread = four rows of one slot
    constexpr int VEC = MEL_ROWS / 4;
    const int m_slot = min(tid / VEC, SEG_SLOTS - 1), m_row = tid % VEC * 4;
    const int m_rem = tid < SEG_SLOTS * VEC && m_row < N_PROJ ? pl.rem[m_slot] : 0;
    const int m_t0 = d.n_steps[m_slot] - m_rem, m_off = m_row / 16 * (SEG_SLOTS * 64) + m_slot * 64 + m_row % 16 * 4;     // [row tile][slot][16 rows]
    int b = 0, b_next = 1;
    for (int s = 0; s < n_steps; ++s) {
        const bool on = s < rem, m_on = s < m_rem;
        if (wave < 4 && on) x.empty4(off_hp(col, g), O_P + b_next * B_P + mt * B_FRAG);
        u32x4_t w = {0u, 0u, 0u, 0u};
        bool in = !m_on;
        for (int spin = 0; spin < x.polls && !in; ++spin) {
            Words::again();
            w = x.look4(m_off, O_M + b * B_M);
            in = m_row == N_MEL ? w.x != EMPTY : Words::full(w);
        }
        stores_done();
        if (m_row == N_MEL || !m_on) w.y = w.z = w.w = 0u;      // no rows beyond the stop row
        if (tid < SEG_SLOTS * VEC) *reinterpret_cast<u32x4_t*>(&s_mel[m_slot][m_row]) = w;
        ps.sync(in);
        {
            uint4 bm[NK3];
#pragma unroll
            for (int f = 0; f < NK3; ++f) bm[f] = *reinterpret_cast<const uint4*>(&s_mel[col][f * KB + g * 4]);
            floatx4 acc[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int f = 0; f < NK3; ++f)
#pragma unroll
                for (int m = 0; m < 2; ++m) acc[m] = mfma_frag<float>(a3[m][f], bm[f], acc[m]);
#pragma unroll
            for (int m = 0; m < 2; ++m)
                *reinterpret_cast<float4*>(&s_hid[col][16 * (wave + 8 * m) + 4 * g]) =
                    make_float4(fmaxf(acc[m][0], 0.f), fmaxf(acc[m][1], 0.f), fmaxf(acc[m][2], 0.f), fmaxf(acc[m][3], 0.f));
        }
        if (ps.bad()) return give_up(d, pl, s);
        lds_barrier();
        if (wave < 4) {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int f = 0; f < NK4; ++f) acc = mfma_frag<float>(a4[f], *reinterpret_cast<const uint4*>(&s_hid[col][f * KB + g * 4]), acc);
            const floatx4 p = {fmaxf(acc[0], 0.f), fmaxf(acc[1], 0.f), fmaxf(acc[2], 0.f), fmaxf(acc[3], 0.f)};
            if (s + 1 < min(rem, n_steps)) x.put4(p, off_hp(col, g), O_P + b * B_P + mt * B_FRAG);
            else if (on) *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(d.xatt[cur ^ ((s + 1) & 1)]) + xoff<float>(NK_A, col, XA_P + 16 * mt + 4 * g)) = p;
        }
        // the books, while the others go on
        if (quarter == 0 && m_on) {
            const size_t at = (size_t)m_slot * d.max_steps + m_t0 + s;
            if (m_row < N_MEL) {
                *reinterpret_cast<u32x4_t*>(d.mel_ring + at * N_MEL + m_row) = w;
                *reinterpret_cast<u32x4_t*>(d.m_last + m_slot * N_MEL + m_row) = w;
            } else {
                d.stop_ring[at] = __uint_as_float(w.x);
                // (no workgroup of this launch reads these two: another LEAD may start after several steps)
                d.t[m_slot] = m_t0 + s + 1;
                if (s + 1 == m_rem) d.done[m_slot] = 1;
            }
        }
        b = b_next;
        b_next = next3(b);
    }
}

// ---------------------------------------------------------------- one request's attention, shared by S workgroups
template <int S>
__device__ __forceinline__ void lsa(const DevPtrs& d, const Words& x, const Pool& pl, int slot, int sp, char* lds, Phases ps)
{
    constexpr int FS = ENC / S, LPR = 64 / S, NA = 4 / S;                  // columns, lanes per row, position classes per lane
    const int cur = pl.cur, n_steps = pl.n_steps;
    const int tid = threadIdx.x, wave = wave_id(), lane = tid & 63, jl = lane & 15, g = lane >> 4;
    float (*s_ctx)[ENC] = reinterpret_cast<float (*)[ENC]>(lds);
    float (*s_u)[U_PAD] = reinterpret_cast<float (*)[U_PAD]>(lds + NW * ENC * 4);
    float* s_e = reinterpret_cast<float*>(s_u + 2);
    float* s_q = s_e + MAX_ENC_LEN;
    float* s_v = s_q + ATT;
    float* s_red = s_v + ATT;
    float (*s_pair)[ATT] = reinterpret_cast<float (*)[ATT]>(s_red + 2 * NW);
    float* s_k = reinterpret_cast<float*>(s_pair + 16);                    // the filters as operands: [filter tile * 16 + channel * 8 + step][lane]
    const int rem = __builtin_amdgcn_readfirstlane(pl.rem[slot]), L = __builtin_amdgcn_readfirstlane(d.L[slot]);
    if (rem == 0) return;
    const int steps = min(rem, n_steps), ntile = (L + 15) >> 4, ML = d.max_enc_len;
    const float* PMs = reinterpret_cast<const float*>(d.PM) + (size_t)slot * ML * ATT + 32 * g;
    // W_loc as in LsaTile<float>: one tile of filters in registers, the other one in LDS
    float4* s_w = reinterpret_cast<float4*>(s_k + 32 * 64);                // [tile of attention dims][lane]
    u32x4_t wA[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) wA[a] = reinterpret_cast<const u32x4_t*>(d.lsa_wfrag)[2 * a * 64 + lane];
    s_w[tid] = reinterpret_cast<const float4*>(d.lsa_wfrag)[(2 * wave + 1) * 64 + lane];
    static_assert(NT == 8 * 64, "a thread a piece");
    for (int i = tid; i < 32 * 64; i += NT) s_k[i] = reinterpret_cast<const float*>(d.lsa_kfrag)[i];
    // the wave's rows of the processed memory of its first tile of positions stay in registers
    u32x4_t pm0[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) pm0[i] = *reinterpret_cast<const u32x4_t*>(PMs + (size_t)min((sp + S * wave) * 16 + jl, L - 1) * ATT + 4 * i);
    // and so do rows of the memory (this workgroup's columns), NP passes of 32 positions; NL more lie in LDS
    constexpr int NP = S == 4 ? 8 : 4, NL = lsa_lds_passes(S);
    const int xw = wave * 4 + lane / LPR * NA;                             // this lane's first position class
    const float* Fslot = reinterpret_cast<const float*>(d.Fmem) + (size_t)slot * ML * ENC;
    const __amdgpu_buffer_rsrc_t f_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Fslot), 0, L * ENC * 4, BUFFER_RSRC_RAW);
    const int f_col = (sp * FS + (lane % LPR) * 8) * 4;
    u32x4_t mem[NP][NA][2];
#pragma unroll
    for (int pp = 0; pp < NP; ++pp)
#pragma unroll
        for (int n = 0; n < NA; ++n)
#pragma unroll
            for (int v = 0; v < 2; ++v) mem[pp][n][v] = __builtin_amdgcn_raw_buffer_load_b128(f_rsrc, (pp * 32 + xw + n) * ENC * 4 + f_col + 16 * v, 0, 0);
    u32x4_t* const s_mem = reinterpret_cast<u32x4_t*>(s_w + 8 * 64) + tid;       // [pass][class][half a row][thread]: the thread's own
    for (int pp = 0; pp < NL && (NP + pp) * 32 < L; ++pp)
#pragma unroll
        for (int i = 0; i < 2 * NA; ++i)
            s_mem[(pp * 2 * NA + i) * NT] = __builtin_amdgcn_raw_buffer_load_b128(f_rsrc, ((NP + pp) * 32 + xw + (i >> 1)) * ENC * 4 + f_col + 16 * (i & 1), 0, 0);
    for (int i = tid; i < ntile * 16 + 32; i += NT) {
        const bool in = i >= LOC_PAD && i < L + LOC_PAD;
        const int jc = min(max(i - LOC_PAD, 0), L - 1);
        s_u[0][i] = in ? d.w_last[cur][(size_t)slot * ML + jc] : 0.f;
        s_u[1][i] = in ? d.w_acc[cur][(size_t)slot * ML + jc] : 0.f;
    }
    if (tid < ATT) s_v[tid] = -2.0f * d.v[tid];
    if (L + tid < ((L + 31) & ~31)) s_e[L + tid] = 0.f;                    // a pass of 32 positions may end past the last
    __syncthreads();
    float vsum = 0.f, bound = 0.f;
#pragma unroll
    for (int at = 0; at < 8; ++at) {
        const float4 vv = *reinterpret_cast<const float4*>(&s_v[32 * g + 4 * at]);
        vsum += (vv.x + vv.y) + (vv.z + vv.w);
    }
    vsum *= -0.5f;
#pragma unroll
    for (int at = 0; at < 8; ++at) {
        const float4 vv = *reinterpret_cast<const float4*>(&s_v[32 * g + 4 * at]);
        bound += (fabsf(vv.x) + fabsf(vv.y)) + (fabsf(vv.z) + fabsf(vv.w));
    }
    bound += __shfl_xor(bound, 16, 64);
    bound += __shfl_xor(bound, 32, 64);
    bound *= 0.5f;
    const bool fast_softmax = bound <= 30.f;

    // loc^T of a tile of 16 positions: the accumulators are the next product's B operands
    struct Loc { floatx4 v[2]; };
    auto loc = [&](int x0) __attribute__((always_inline)) {
        Loc l = {{floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}}};
#pragma unroll
        for (int cs = 0; cs < 16; ++cs) {
            const float u = s_u[cs >> 3][x0 + g + 4 * (cs & 7)];
#pragma unroll
            for (int m = 0; m < 2; ++m) l.v[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(s_k[(m * 16 + cs) * 64 + lane], u, l.v[m], 0, 0, 0);
        }
        return l;
    };
    // the energies of one workgroup's tiles lie together: [workgroup][its tiles][16 positions]
    const int e_slot = segment_energy_bytes(ML);
    auto e_off = [&](int j) { return (j >> 4) % S * (e_slot / S) + (j >> 4) / S * 64 + (j & 15) * 4; };
    // this thread's share of the query: four rows of two of its 32 partial products
    const int q_off = (tid >> 5) * 2 * ATT * 4 + (tid & 31) * 16, b_e = SEG_SLOTS * e_slot, e_at = O_E + slot * e_slot;
    const int k_a = sp * FS + tid, a_off = slot * (ENC * 4) + k_a * 4;
    int b = 0, b_next = 1;
    for (int s = 0; s < steps; ++s) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            keep(pm0[i]);
            keep(wA[i]);
        }
#pragma unroll
        for (int i = 0; i < NP * NA * 2; ++i) keep(mem[i / (2 * NA)][i / 2 % NA][i & 1]);
        for (int tt = sp + S * wave; tt < ntile; tt += S * NW)
            if (g == 0 && tt * 16 + jl < L) x.empty(e_off(tt * 16 + jl), e_at + b_next * b_e);
        if (tid < FS) x.empty(a_off, O_A + b_next * B_A);
        // the location features do not wait for the query
        const Loc loc0 = loc(min((sp + S * wave) * 16, (ntile - 1) * 16) + jl);
        {
            u32x4_t w0, w1;
            bool in = false;
            for (int spin = 0; spin < x.polls && !in; ++spin) {
                Words::again();
                w0 = x.look4(q_off, O_Q + b * B_Q + slot * B_QS);
                w1 = x.look4(q_off + ATT * 4, O_Q + b * B_Q + slot * B_QS);
                in = Words::full(w0) && Words::full(w1);
            }
            stores_done();
            floatx4 p;
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = __uint_as_float(w0[i]) + __uint_as_float(w1[i]);
            *reinterpret_cast<floatx4*>(&s_pair[tid >> 5][(tid & 31) * 4]) = p;
            ps.sync(in);
        }
        if (tid < ATT) {
            float sq[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                sq[h] = s_pair[4 * h][tid];
#pragma unroll
                for (int i = 1; i < 4; ++i) sq[h] += s_pair[4 * h + i][tid];
            }
            s_q[tid] = (sq[0] + sq[1]) + (sq[2] + sq[3]);
        }
        if (ps.bad()) return lose_one(d, slot);
        lds_barrier();
        auto energies = [&](int tt, const u32x4_t (&pm)[8], const Loc& l) __attribute__((always_inline)) {
            const int j = tt * 16 + jl;
            float e = vsum;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                floatx4 p[4];
#pragma unroll
                for (int a = 0; a < 4; ++a) p[a] = *reinterpret_cast<const floatx4*>(&s_q[32 * g + 16 * half + 4 * a]);
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    u32x4_t w[4];
#pragma unroll
                    for (int a = 0; a < 4; ++a) w[a] = m == 0 ? wA[4 * half + a] : *reinterpret_cast<const u32x4_t*>(&s_w[(4 * half + a) * 64 + lane]);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int a = 0; a < 4; ++a) p[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[a][i]), l.v[m][i], p[a], 0, 0, 0);
                }
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const float4 vv = *reinterpret_cast<const float4*>(&s_v[32 * g + 16 * half + 4 * a]);
                    const u32x4_t& u = pm[4 * half + a];
                    e = fmaf(vv.x, half_one_minus_tanh(p[a][0] + __uint_as_float(u.x)), e);
                    e = fmaf(vv.y, half_one_minus_tanh(p[a][1] + __uint_as_float(u.y)), e);
                    e = fmaf(vv.z, half_one_minus_tanh(p[a][2] + __uint_as_float(u.z)), e);
                    e = fmaf(vv.w, half_one_minus_tanh(p[a][3] + __uint_as_float(u.w)), e);
                }
            }
            e += xor16(e);
            e += xor32(e);
            if (fast_softmax) e = __expf(e - bound);
            if (g == 0 && j < L) {
                s_e[j] = e;
                x.put(__float_as_uint(e), e_off(j), e_at + b * b_e);
            }
        };
        if (sp + S * wave < ntile) energies(sp + S * wave, pm0, loc0);
        for (int tt = sp + S * (wave + NW); tt < ntile; tt += S * NW) {        // longer texts: from memory
            u32x4_t pm[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) pm[i] = *reinterpret_cast<const u32x4_t*>(PMs + (size_t)min(tt * 16 + jl, L - 1) * ATT + 4 * i);
            energies(tt, pm, loc(tt * 16 + jl));
        }
        bool ok = true;
        for (int i = tid; i < L; i += NT) {
            if ((i >> 4) % S == sp) continue;
            unsigned w = 0u;
            bool in = false;
            for (int spin = 0; spin < x.polls && !in; ++spin) {
                Words::again();
                w = x.look(e_off(i), e_at + b * b_e);
                in = w != EMPTY;
            }
            ok = ok && in;
            s_e[i] = __uint_as_float(w);
        }
        stores_done();
        ps.sync(ok);
        float psum = 0.f;
        for (int tt = wave; tt < ntile; tt += NW) {
            const int j = tt * 16 + jl;
            if (g == 0 && j < L) psum += s_e[j];
        }
        psum = wave_sum_fast(psum);
        if (lane == 0) s_red[NW + wave] = psum;                            // read behind the barrier of the context's sums
        if (ps.bad()) return lose_one(d, slot);
        if (!fast_softmax) {
            float mx = -INFINITY;
            for (int i = tid; i < L; i += NT) mx = fmaxf(mx, s_e[i]);
            mx = wave_max(mx);
            if (lane == 0) s_red[wave] = mx;
            lds_barrier();
            mx = s_red[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) mx = fmaxf(mx, s_red[w]);
            float sum = 0.f;
            for (int i = tid; i < L; i += NT) {
                const float p = __expf(s_e[i] - mx);
                s_e[i] = p;
                sum += p;
            }
            sum = wave_sum(sum);
            if (lane == 0) s_red[NW + wave] = sum;
            lds_barrier();
        }

        float acc[NA][8];
#pragma unroll
        for (int n = 0; n < NA; ++n)
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[n][i] = 0.f;
        auto add = [&](int n, int px, const u32x4_t (&r)[2]) __attribute__((always_inline)) {
            const float w = s_e[px];
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[n][i] = fmaf(w, __uint_as_float(r[i >> 2][i & 3]), acc[n][i]);
        };
#pragma unroll
        for (int pp = 0; pp < NP; ++pp) {
            if (pp * 32 >= L) break;
#pragma unroll
            for (int n = 0; n < NA; ++n) add(n, pp * 32 + xw + n, mem[pp][n]);
        }
#pragma unroll 1
        for (int pp = NP; pp < NP + NL && pp * 32 < L; ++pp)
#pragma unroll
            for (int n = 0; n < NA; ++n) {
                const u32x4_t r[2] = {s_mem[((pp - NP) * 2 * NA + 2 * n) * NT], s_mem[((pp - NP) * 2 * NA + 2 * n + 1) * NT]};
                add(n, pp * 32 + xw + n, r);
            }
        constexpr int MORE = 4 / NA;
        for (int x0 = 32 * (NP + NL); x0 < L; x0 += 32 * MORE) {                  // longer texts: from memory
            u32x4_t more[MORE][NA][2];
#pragma unroll
            for (int pp = 0; pp < MORE; ++pp)
#pragma unroll
                for (int n = 0; n < NA; ++n)
#pragma unroll
                    for (int v = 0; v < 2; ++v) more[pp][n][v] = __builtin_amdgcn_raw_buffer_load_b128(f_rsrc, (x0 + pp * 32 + xw + n) * ENC * 4 + f_col + 16 * v, 0, 0);
#pragma unroll
            for (int pp = 0; pp < MORE; ++pp)
                if (x0 + pp * 32 < L)
#pragma unroll
                    for (int n = 0; n < NA; ++n) add(n, x0 + pp * 32 + xw + n, more[pp][n]);
        }
        // (classes held by one lane are paired here)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float t = acc[0][i];
            if constexpr (NA >= 2) t = acc[0][i] + acc[1][i];
            s_ctx[wave][lane * 8 + i] = t;
        }
        lds_barrier();
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += s_red[NW + w];
        const float inv = 1.0f / sum;
        if (tid < FS) {
            float c = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                float t = s_ctx[w][tid] + s_ctx[w][LPR * 8 + tid];
                if constexpr (S == 4) t += s_ctx[w][2 * LPR * 8 + tid] + s_ctx[w][3 * LPR * 8 + tid];
                c += t;
            }
            const float a = c * inv;
            x.put(__float_as_uint(a), a_off, O_A + b * B_A);
            if (s + 1 == steps) {
                const int end = cur ^ (steps & 1);
                reinterpret_cast<float*>(d.xatt[end])[xoff<float>(NK_A, slot, XA_A + k_a)] = a;
                reinterpret_cast<float*>(d.xdec[end ^ 1])[xoff<float>(NK_D, slot, XD_A + k_a)] = a;
            }
        }
        // the new weights: every workgroup of the request keeps all of them
        for (int i = tid; i < L; i += NT) {
            const float w = s_e[i] * inv;
            s_u[0][i + LOC_PAD] = w;
            s_u[1][i + LOC_PAD] += w;
        }
        lds_barrier();
        b = b_next;
        b_next = next3(b);
    }
    const int end = cur ^ (steps & 1);
    for (int i = sp + S * tid; i < L; i += S * NT) {
        d.w_last[end][(size_t)slot * ML + i] = s_u[0][i + LOC_PAD];
        d.w_acc[end][(size_t)slot * ML + i] = s_u[1][i + LOC_PAD];
    }
}

// Which workgroup does what: GATES on all XCDs, ATT on 0 .. 3, LSA on 4 .. 7 (a request's on one), the projection and its leaders beside
// ATT.  Five CUs or more of every XCD stay free for work on other streams.
constexpr int WGS = 27;                                     // on an XCD
template <int S>
__global__ __launch_bounds__(NT) void k_segment32(DevPtrs d, int cur, int n_slots, int n_steps, char* words, char* words_next, int bytes, int empty_bytes, SegmentLeft left)
{
    __shared__ __attribute__((aligned(16))) char lds[S_MAX];
    __shared__ int s_failed, s_rem[SEG_SLOTS];
    if (threadIdx.x == 0) s_failed = 0x7fffffff;
    if (threadIdx.x < SEG_SLOTS) {
        const int sl = threadIdx.x;
        s_rem[sl] = sl < n_slots ? segment_left(d, left, sl) : 0;
    }
    for (int at = (blockIdx.x * NT + threadIdx.x) * 16; at < empty_bytes; at += gridDim.x * NT * 16)
        *reinterpret_cast<u32x4_t*>(words_next + at) = u32x4_t{EMPTY, EMPTY, EMPTY, EMPTY};
    __syncthreads();
    const Phases ps = {&s_failed};
    const Pool pl = {cur, n_steps, 1, bytes, s_rem};
    const Words x = {words, bytes, d.wait_polls};
    const int xcd = blockIdx.x & 7, i = blockIdx.x >> 3, k = i - GATES / 8;
    if (k < 0) {
        gates(d, x, pl, xcd * (GATES / 8) + i, lds, ps);
    } else if (xcd >= 4) {
        const int slot = k / S * 4 + xcd - 4;
        if (k < 8 && slot < n_slots) lsa<S>(d, x, pl, slot, k % S, lds, ps);
    } else if (k < 8) {
        att(d, x, pl, xcd * 8 + k, lds, ps);
    } else if (xcd < 2) {
        rows(d, x, pl, xcd * 3 + k - 8, lds, ps);
    } else if (k < 10) {
        lead(d, x, pl, (xcd - 2) * 2 + k - 8, lds, ps);
    }
}

}  // namespace

hipError_t launch_segment32(const DevPtrs& d, int cur, int n_slots, int n_steps, int set, int empty_tiles, const SegmentLeft& left, hipStream_t s)
{
    if (!d.seg_x || n_slots < 1 || n_slots > SEG_SLOTS || n_steps < 1 || (set & ~1) || (empty_tiles & ~1) || d.stop_threshold >= 0.f) return hipErrorInvalidValue;
    const size_t bytes = segment32_bytes(d.max_enc_len);
    char* words = static_cast<char*>(d.seg_x);
    static_assert(HID / 8 == GATES && GATES / 8 + 8 + 3 == WGS && 4 * 8 >= 2 * SEG_SLOTS, "eight units a GATES; ATT, LSA and the projection beside them");
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(8 * WGS), dim3(NT), 0, s, d, cur, n_slots, n_steps, words + set * bytes, words + (set ^ 1) * bytes, (int)bytes,
                           (int)(empty_tiles * bytes), left);
    };
    if (n_slots <= 8) go(k_segment32<4>);
    else go(k_segment32<2>);
    return hipGetLastError();
}

}  // namespace tts
