// A segment of decoder steps as ONE launch, for two-byte pools whose running requests lie in the first SEG_TILES tiles of 16 slots.
//
// What bounds a step of so small a pool is a chain: p -> attention LSTM -> query -> energies -> context -> decoder LSTM -> frame
// -> p.  As launches of its own (k_lsa, k_proj) a step takes 16.8 us at one request, 6 us of it two launch boundaries with the
// start-up and the first cold round trips behind them, and every launch pulls its share of the 36 MB of weights again.  Here the
// workgroups stay for the whole segment: each keeps its part of the weights in registers and LDS and its part of the requests'
// state in registers, and the links of the chain are words handed from workgroup to workgroup through memory.  One such hop takes
// 0.4 to 0.6 us from store to seen (64 words handed to and fro between two workgroups, on one XCD or on different ones).
//
// Workgroups (eight waves, one per CU; blockIdx % 8 is the XCD), and what each does in step s:
//   32 x ATT   32 hidden units of the attention LSTM each: gates from p (K = 256) and the pre-sums, cell, h and the units' rank-32
//              share of the query out; then, off the chain, the gate pre-sums of step s + 1 from a and h_att
//   S x LSA    per request, on one XCD: energies shared among the S, softmax, a share of the context's columns each; the
//              attention weights stay in LDS, the rows of the request's memory (up to 512 positions) in registers
//   64 x DEC   16 hidden units of the decoder LSTM each: the sums over h_dec and h_att ahead of the chain, those over a on it
//   per tile: 6 x ROWS   one row tile of the projection each; 1 x LEAD: frame, prenet, books
// ATT and DEC serve the tiles one after the other; one tile is bound by the chain, three by the work of an ATT.
// Every product and every sum is formed in the order of the kernels in kernels.hip, so a request's frames and state are the
// same bits whichever form a step takes.
//
// A word is its own flag: a buffer is filled with EMPTY, a pattern no value is stored as, and a reader polls until none of its
// words is EMPTY.  Each kind of word has three buffers, step s's is s % 3, and a workgroup empties its words of buffer (s + 1) % 3
// (ATT: of buffer (s + 2) % 3, at the end of its step) before it stores those of step s (s + 1):
//   * the readers of step s - 2's words, which lay there, are done: the workgroup has seen words that could not have been made
//     before all of them were (each role's readers lie on the chain of step s - 1, which led to what it has received in step s);
//   * a reader of step s + 1 finds them emptied: it has taken this workgroup's words of step s, which were stored after the
//     emptying had been acknowledged (a poll that the storing wave has waited for lies in between).
// A launch uses one of two such sets and empties the other one, whole, before it waits for anything: the next launch finds its set
// empty whatever became of this one.
// Every wait is bounded; a workgroup whose wait runs out marks the requests that take part in the step as ended and failed (LSA: its own, and
// those that wait for its part of a then mark the others), stores nothing more and leaves, and the others' waits run out in turn.  So one
// workgroup that other work keeps from starting for the length of a wait ends every request of the step, where the step's launches end one
// request (k_lsa) or a tile of them (k_proj).  The workgroups of a segment all have to be resident: other pools' launches are kept away
// (resident.h), work that ends by itself delays them.
#include "kernels.h"
#include "lsa_tile.h"
#include "mfma.h"
#include "segment_parts.h"
#include "words.h"

namespace tts {
namespace {

constexpr int KB = Frag<h16_t>::KB;
constexpr int NK_A = K_ATT / KB, NK_D = K_DEC / KB, NK_P = K_PROJ / KB;    // fragments per row tile: 56, 80, 48
constexpr int F_H = HID / KB, F_A = ENC / KB, F_P = PRENET / KB;            // fragments of h, a, p: 32, 16, 8
static_assert(F_H == 4 * NW && F_A == 2 * NW && F_P == NW, "a wave takes four fragments of h, two of a, one of p");
constexpr int MEL_ROWS = 96;

// One buffer of each kind, in bytes.  What one workgroup (for q and p: one wave) stores lies together, a request's share of it in whole
// 32 to 512 bytes: polls are L2 hits (0.12 us a round of 8 KB) until somebody stores to the line, which the XCD then takes from memory
// anew, so a line that fills in many small steps is fetched many times.  With words of several workgroups in a line (all in B-operand
// order, stored as they were made, 4 bytes a lane) a step took 10.6 us at 1 request, 13.7 at 8 and 17.4 at 16; like this 9.7, 10.7, 12.1.
constexpr int B_FRAG = 1024, B_H = F_H * B_FRAG, B_A = F_A * B_FRAG, B_P = F_P * B_FRAG;
constexpr int B_QS = QUERY_PARTIALS * ATT * 4, B_Q = SEG_SLOTS * B_QS, B_M = SEG_SLOTS * MEL_ROWS * 4;
constexpr int O_HA = 0, O_HD = O_HA + 3 * B_H, O_A = O_HD + 3 * B_H, O_P = O_A + 3 * B_A, O_Q = O_P + 3 * B_P, O_M = O_Q + 3 * B_Q, O_E = O_M + 3 * B_M;
static_assert(O_E == SEG_FIXED_BYTES, "the arena's share");

// a lane's offset in a fragment: of h_att and p ([fragment][slot][32 halves]), of h_dec ([half a fragment][slot][16 halves]: one of the
// decoder LSTM's workgroups stores half a fragment) and of a ([slot][512 halves])
__device__ __forceinline__ int off_hp(int col, int g) { return col * 64 + g * 16; }
__device__ __forceinline__ int off_hd(int col, int g) { return ((g >> 1) * SEG_SLOTS + col) * 32 + (g & 1) * 16; }
__device__ __forceinline__ int off_a(int col, int g) { return col * (ENC * 2) + g * 16; }

constexpr int ATT_LDS_RT = 2;                               // row tiles whose late fragments lie in LDS: registers hold six
constexpr int ATT_LATE = 6;                                 // late fragments per wave and row tile: two of a, four of h_att
constexpr int S_ATT_W = ATT_LDS_RT * ATT_LATE * NW * 1024, S_ATT_RED = NW * 4 * 1024, S_ATT_B = F_P * 1024;
constexpr int S_ATT = S_ATT_W + S_ATT_RED + S_ATT_B + 32 * 16 * 4 + 16 * 32 * 2;
constexpr int S_DEC_RED = 2 * NW * 4 * 1024, S_DEC_W = NW * 7 * 1024;
constexpr int S_DEC_PRE = SEG_TILES * 2 * 256 * 16, S_DEC_RED2 = NW * 4 * 1024;            // several tiles, one tile: in the same place
constexpr int S_DEC = S_DEC_RED + S_DEC_W + (S_DEC_PRE > S_DEC_RED2 ? S_DEC_PRE : S_DEC_RED2);
constexpr int P_LD = 68;                                    // the reduction reads 4 columns x 16 rows a wave: a bank each
constexpr int S_ROWS = 6 * NW * 4 * P_LD * 4;
constexpr int MEL_LD = MEL_ROWS + 8, HID_LD = PRENET + 8;     // halves: an odd number of 16-byte pieces a row
constexpr int S_LEAD = 16 * (MEL_LD + HID_LD) * 2;
constexpr int U_PAD = MAX_ENC_LEN + 48;
constexpr int S_LSA = (NW * ENC + 16 * ATT + 2 * U_PAD + MAX_ENC_LEN + 2 * ATT + 2 * NW) * 4;
constexpr int S_MAX = S_DEC;
static_assert(S_ATT <= S_MAX && S_ROWS <= S_MAX && S_LEAD <= S_MAX && S_LSA <= S_MAX && S_MAX + 64 <= 160 * 1024, "the roles' LDS");

// ---------------------------------------------------------------- the attention LSTM and the query
// MULTI: more tiles than one.  The cells and the pre-sums then live in memory from step to step (each thread's own words of the arrays
// the step kernels use: requested ahead of the wait for p), else in registers.
template <bool MULTI>
__device__ __forceinline__ void seg_att(const DevPtrs& d, const Words& words, const Pool& pl, int rg, char* lds, Phases ps)
{
    const int wave = wave_id(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4, cur = pl.cur, n_steps = pl.n_steps;
    const int rt = rg * 8 + wave, unit = rt * 4 + g;
    uint4* s_w = reinterpret_cast<uint4*>(lds);                                             // [2][6 f][8 waves][64]
    floatx4 (*red)[4][64] = reinterpret_cast<floatx4 (*)[4][64]>(lds + S_ATT_W);
    uint4 (*s_b)[64] = reinterpret_cast<uint4 (*)[64]>(lds + S_ATT_W + S_ATT_RED);
    float (*s_h)[16] = reinterpret_cast<float (*)[16]>(lds + S_ATT_W + S_ATT_RED + S_ATT_B);
    h16_t (*s_hh)[32] = reinterpret_cast<h16_t (*)[32]>(s_h + 32);                          // [slot][unit]

    uint4 we[F_P], wl[8 - ATT_LDS_RT][ATT_LATE];
#pragma unroll
    for (int f = 0; f < F_P; ++f) we[f] = d.Wa[xfrag(NK_A, rt, f, lane)];
#pragma unroll
    for (int r = 0; r < 8 - ATT_LDS_RT; ++r)
#pragma unroll
        for (int f = 0; f < ATT_LATE; ++f) wl[r][f] = d.Wa[xfrag(NK_A, rg * 8 + r, wave + 8 * (f + 1), lane)];
#pragma unroll
    for (int r = 0; r < ATT_LDS_RT; ++r)
#pragma unroll
        for (int f = 0; f < ATT_LATE; ++f)
            s_w[((r * ATT_LATE + f) * NW + wave) * 64 + lane] = d.Wa[xfrag(NK_A, rg * 8 + 8 - ATT_LDS_RT + r, wave + 8 * (f + 1), lane)];
    float wq[8];                                            // W_q[16 wave + ..][32 rg + 4 k + ..]
#pragma unroll
    for (int k = 0; k < 8; ++k) wq[k] = d.Wq_epi[((size_t)(rg * 8 + k) * 8 + wave) * 64 + lane];
    const floatx4 bias4 = *reinterpret_cast<const floatx4*>(d.ba + unit * 4);
    floatx4* pre_g = reinterpret_cast<floatx4*>(d.pre_att) + (size_t)rt * 64 + lane;
    float* c_g = d.c_att + (size_t)col * HID + unit;
    constexpr int PRE_TILE = HID / 4 * 64, C_TILE = 16 * HID, NAP = MULTI ? 4 : 16;
    floatx4 pre4 = pre_g[0];
    float c = c_g[0];
    const int q_off = col * B_QS + (16 * wave + 4 * g) * 4;

    int b = 0, b_before = 2, b_next = 1;
    for (int s = 0; s < n_steps; ++s) {
        // Several tiles: what tile t + 1 needs is asked for while tile t's gates are formed and is there before tile t's words are stored
        // (loads return in the order of the requests: behind a store they would wait for its acknowledgement).
        u32x4_t p_next[1];
        floatx4 pre_next = pre4;
        float c_next = c;
        auto ask = [&](int t) __attribute__((always_inline)) {
            if (s > 0) words.of(t, pl.tile_bytes).ahead<1, B_FRAG>(O_P + b_before * B_P, wave, off_hp(col, g), p_next);
            else p_next[0] = reinterpret_cast<const u32x4_t*>(d.xatt[cur])[xfrag(NK_A, t, wave, lane)];
            pre_next = pre_g[t * PRE_TILE];
            c_next = c_g[t * C_TILE];
        };
        if constexpr (MULTI) {
            ask(0);
            stores_done();                                  // (and all tiles' emptying, in the step before)
        }
        for (int t = 0; t < (MULTI ? pl.n_tiles : 1); ++t) {
            const Words x = words.of(t, pl.tile_bytes);
            const int rem = pl.rem[t * 16 + col];
            const bool on = s < rem;
            bool ok = true;
            uint4 pb[1];
            if constexpr (MULTI) {
                pre4 = pre_next;
                c = c_next;
                if (s > 0) ok = x.take_rest<1, B_FRAG>(O_P + b_before * B_P, wave, off_hp(col, g), on, p_next, pb);
                else pb[0] = as_uint4(p_next[0]);
            } else {
                if (s > 0) ok = x.take<1, B_FRAG>(O_P + b_before * B_P, wave, off_hp(col, g), on, pb);
                else pb[0] = reinterpret_cast<const uint4*>(d.xatt[cur])[xfrag(NK_A, t, wave, lane)];
                stores_done();
            }
            s_b[wave][lane] = pb[0];
            ps.sync(ok);
            if constexpr (MULTI) ask(min(t + 1, pl.n_tiles - 1));
            floatx4 g4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int f = 0; f < F_P; ++f) g4 = mfma_frag<h16_t>(we[f], s_b[f][lane], g4);
            g4 += bias4;
            g4 += pre4;
            float c_new = c, hf;
            cell(g4, c_new, hf);
            const h16_t h = from_float<h16_t>(hf);
            s_h[4 * wave + g][col] = on ? to_float(h) : 0.f;
            s_hh[col][4 * wave + g] = h;
            if (ps.bad()) return give_up(d, pl, s);
            lds_barrier();
            // the units' share of the query: 16 rows per wave
            {
                floatx4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 8; ++k) part = __builtin_amdgcn_mfma_f32_16x16x4f32(wq[k], s_h[4 * k + g][col], part, 0, 0, 0);
                if constexpr (MULTI) stores_done();
                if (on) x.put4(part, q_off, O_Q + b * B_Q + rg * ATT * 4);
                if (wave == 0 && on) x.put4(*reinterpret_cast<const floatx4*>(&s_hh[col][8 * g]), off_hp(col, g), O_HA + b * B_H + rg * B_FRAG);
            }
            const bool last = s + 1 == min(rem, n_steps);
            if (on) c = c_new;
            if (MULTI ? on : last) c_g[t * C_TILE] = c;
            if (last) {
                // the request's last step of this segment: its state where the step kernels keep it
                const int end = cur ^ ((s + 1) & 1);
                reinterpret_cast<h16_t*>(d.xatt[end])[xoff<h16_t>(NK_A, t * 16 + col, XA_H + unit)] = h;
                reinterpret_cast<h16_t*>(d.xdec[end ^ 1])[xoff<h16_t>(NK_D, t * 16 + col, XD_HA + unit)] = h;
            }
        }

        // off the chain: the next step's gate pre-sums over [a; h_att]
        for (int t = 0; t < (MULTI ? pl.n_tiles : 1); ++t) {
            const Words x = words.of(t, pl.tile_bytes);
            const bool on = s < pl.rem[t * 16 + col];
            uint4 hb[4], ab[2];
            // (a comes last: by then the larger h_att has been asked for once)
            bool ok;
            if constexpr (MULTI) {
                u32x4_t h_look[4];
                x.ahead<4, B_FRAG>(O_HA + b * B_H, wave, off_hp(col, g), h_look);
                ok = x.take<2, 64, NAP>(O_A + b * B_A, wave, off_a(col, g), on, ab);
                ok = x.take_rest<4, B_FRAG, NAP>(O_HA + b * B_H, wave, off_hp(col, g), on, h_look, hb) && ok;
            } else {
                ok = x.take<2, 64, NAP>(O_A + b * B_A, wave, off_a(col, g), on, ab);
                ok = x.take<4, B_FRAG, NAP>(O_HA + b * B_H, wave, off_hp(col, g), on, hb) && ok;
            }
            // (step s - 1's words, whose buffer is step s + 2's: taken before this step's a was made)
            if (wave == 0 && on) x.empty4(off_hp(col, g), O_HA + b_before * B_H + rg * B_FRAG);
            if (on) x.empty4(q_off, O_Q + b_before * B_Q + rg * ATT * 4);
            if (MULTI && t > 0) lds_barrier();
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (half) lds_barrier();
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int r = 4 * half + r4;
                    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int f = 0; f < ATT_LATE; ++f) {
                        const uint4 w = r < 8 - ATT_LDS_RT ? wl[r < 8 - ATT_LDS_RT ? r : 0][f]
                                                           : s_w[(((r - (8 - ATT_LDS_RT)) * ATT_LATE + f) * NW + wave) * 64 + lane];
                        acc = mfma_frag<h16_t>(w, f < 2 ? ab[f < 2 ? f : 0] : hb[f < 2 ? 0 : f - 2], acc);
                    }
                    red[wave][r4][lane] = acc;
                }
                if (half) lds_barrier();
                else ps.sync(ok);
                if (wave >> 2 == half) {
                    pre4 = red[0][wave & 3][lane];
#pragma unroll
                    for (int w = 1; w < NW; ++w) pre4 += red[w][wave & 3][lane];
                }
            }
            if (ps.bad()) return give_up(d, pl, s);
            if (MULTI || s + 1 == n_steps) pre_g[t * PRE_TILE] = pre4;
        }
        b_before = b;
        b = b_next;
        b_next = next3(b);
    }
}

// ---------------------------------------------------------------- the decoder LSTM
template <bool MULTI>
__device__ __forceinline__ void seg_dec(const DevPtrs& d, const Words& words, const Pool& pl, int j, char* lds, Phases ps)
{
    const int wave = wave_id(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4, cur = pl.cur, n_steps = pl.n_steps;
    // reduction buffers in turn: what was read from one is done when the barrier of the other has been passed (one tile: a third one,
    // where several tiles keep the sums over h, saves a barrier)
    floatx4 (*red0)[4][64] = reinterpret_cast<floatx4 (*)[4][64]>(lds);
    floatx4 (*red1)[4][64] = red0 + NW;
    floatx4 (*red2)[4][64] = reinterpret_cast<floatx4 (*)[4][64]>(lds + S_DEC_RED + S_DEC_W);
    uint4* s_w = reinterpret_cast<uint4*>(lds + S_DEC_RED) + wave * 7 * 64 + lane;              // [wave][7][64]: the wave's own
    floatx4* s_pre = reinterpret_cast<floatx4*>(lds + S_DEC_RED + S_DEC_W) + threadIdx.x;       // [tile][h_dec, h_att][256 threads]
    uint4 w[4][NK_D / NW];                                  // fragments wave + 8 f: h_att (f = 0 .. 3), a (4, 5), h_dec (6 .. 9)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int f = 0; f < NK_D / NW; ++f)
            if (r < 3 || f == 0 || f == 4 || f == 5) w[r][f] = d.Wd[xfrag(NK_D, 4 * j + r, wave + 8 * f, lane)];
#pragma unroll
    for (int f = 0; f < 7; ++f) s_w[f * 64] = d.Wd[xfrag(NK_D, 4 * j + 3, wave + 8 * (f < 3 ? f + 1 : f + 3), lane)];   // registers hold the others
    const int er = wave & 3, rt = 4 * j + er, unit = rt * 4 + g, hd_off = col * 32 + er * 8 + (g >> 1) * 4;
    const floatx4 bias4 = *reinterpret_cast<const floatx4*>(d.bd + unit * 4);
    float* c_g = d.c_dec + (size_t)col * HID + unit;
    constexpr int C_TILE = 16 * HID, NAP = MULTI ? 2 : 8;
    float c = c_g[0];

    int b = 0, b_before = 2, b_next = 1;
    for (int s = 0; s < n_steps; ++s) {
        floatx4 pre4, pre4b;
        // ahead of the chain: the sums over h_dec of the step before (all tiles') and over h_att
        auto over_hd = [&](int t, floatx4 (*red)[4][64]) __attribute__((always_inline)) {
            const Words x = words.of(t, pl.tile_bytes);
            const bool on = s < pl.rem[t * 16 + col];
            bool ok = true;
            uint4 hd[4];
            if (s > 0) {
                ok = x.take<4, B_FRAG, NAP>(O_HD + b_before * B_H, wave, off_hd(col, g), on, hd);
            } else {
#pragma unroll
                for (int f = 0; f < 4; ++f) hd[f] = reinterpret_cast<const uint4*>(d.xdec[cur])[xfrag(NK_D, t, XD_HD / KB + wave + 8 * f, lane)];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < 4; ++f) acc = mfma_frag<h16_t>(r < 3 ? w[r][6 + f] : s_w[(3 + f) * 64], hd[f], acc);
                red[wave][r][lane] = acc;
            }
            return ok;
        };
        auto over_ha = [&](int t, floatx4 (*red)[4][64]) __attribute__((always_inline)) {
            const Words x = words.of(t, pl.tile_bytes);
            uint4 ha[4];
            const bool ok = x.take<4, B_FRAG, NAP>(O_HA + b * B_H, wave, off_hp(col, g), s < pl.rem[t * 16 + col], ha);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < 4; ++f) acc = mfma_frag<h16_t>(r < 3 || f == 0 ? w[r][f] : s_w[(f - 1) * 64], ha[f], acc);
                red[wave][r][lane] = acc;
            }
            return ok;
        };
        auto sum = [&](floatx4 (*red)[4][64]) __attribute__((always_inline)) {
            floatx4 v = red[0][er][lane];
#pragma unroll
            for (int k = 1; k < NW; ++k) v += red[k][er][lane];
            return v;
        };
        if constexpr (MULTI) {
            for (int i = 0; i < 2 * pl.n_tiles; ++i) {
                const int t = i < pl.n_tiles ? i : i - pl.n_tiles;
                floatx4 (*red)[4][64] = i & 1 ? red1 : red0;
                ps.sync(i < pl.n_tiles ? over_hd(t, red) : over_ha(t, red));
                const floatx4 v = sum(red);
                if (ps.bad()) return give_up(d, pl, s);
                if (wave < 4) s_pre[(2 * t + (i < pl.n_tiles ? 0 : 1)) * 256] = v;
                // (h_att has come: see the top of the file)
                if (i >= pl.n_tiles && wave < 4 && !(g & 1) && s < pl.rem[t * 16 + col])
                    words.of(t, pl.tile_bytes).empty(hd_off, O_HD + b_next * B_H + j * (B_FRAG / 2));
            }
        } else {
            bool ok = over_hd(0, red0);
            ok = over_ha(0, red1) && ok;
            ps.sync(ok);
            pre4 = sum(red0);
            pre4b = sum(red1);
            if (ps.bad()) return give_up(d, pl, s);
        }

        // (several tiles: asked for ahead, as in the attention LSTM)
        u32x4_t a_next[2];
        float c_next = c;
        auto ask = [&](int t) __attribute__((always_inline)) {
            words.of(t, pl.tile_bytes).ahead<2, 64>(O_A + b * B_A, wave, off_a(col, g), a_next);
            c_next = c_g[t * C_TILE];
        };
        if constexpr (MULTI) {
            ask(0);
            stores_done();
        }
        for (int t = 0; t < (MULTI ? pl.n_tiles : 1); ++t) {
            const Words x = words.of(t, pl.tile_bytes);
            const int rem = pl.rem[t * 16 + col];
            const bool on = s < rem;
            floatx4 (*red)[4][64] = !MULTI ? red2 : t & 1 ? red1 : red0;
            if constexpr (MULTI) c = c_next;
            else if (wave < 4 && on && !(g & 1)) x.empty(hd_off, O_HD + b_next * B_H + j * (B_FRAG / 2));
            uint4 ab[2];
            bool ok;
            if constexpr (MULTI) {
                ok = x.take_rest<2, 64>(O_A + b * B_A, wave, off_a(col, g), on, a_next, ab);
                ask(min(t + 1, pl.n_tiles - 1));
            } else {
                ok = x.take<2, 64>(O_A + b * B_A, wave, off_a(col, g), on, ab);
                stores_done();
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma_frag<h16_t>(w[r][4], ab[0], acc);
                acc = mfma_frag<h16_t>(w[r][5], ab[1], acc);
                red[wave][r][lane] = acc;
            }
            ps.sync(ok);
            floatx4 g4 = bias4;
#pragma unroll
            for (int k = 0; k < NW; ++k) g4 += red[k][er][lane];
            if constexpr (MULTI) {
                pre4 = s_pre[(2 * t) * 256 - (wave & 4) * 64];
                pre4b = s_pre[(2 * t + 1) * 256 - (wave & 4) * 64];
            }
            g4 += pre4;
            g4 += pre4b;
            float c_new = c, hf;
            cell(g4, c_new, hf);
            const h16_t h = from_float<h16_t>(hf);
            if (ps.bad()) return give_up(d, pl, s);
            // (waves 4 .. 7 form the same cells and store nothing)
            // units 0, 1 and 2, 3 of a column in one word: the lanes of odd units hand theirs to the lanes before them
            const auto sw = __builtin_amdgcn_permlane16_swap((unsigned)h.bits, (unsigned)h.bits, false, false);
            if constexpr (MULTI) stores_done();
            if (wave < 4 && on && !(g & 1)) x.put(sw[0] | sw[1] << 16, hd_off, O_HD + b * B_H + j * (B_FRAG / 2));
            const bool last = s + 1 == min(rem, n_steps);
            if (on) c = c_new;
            if (wave < 4 && (MULTI ? on : last)) c_g[t * C_TILE] = c;
            if (wave < 4 && last)
                reinterpret_cast<h16_t*>(d.xdec[cur ^ ((s + 1) & 1)])[xoff<h16_t>(NK_D, t * 16 + col, XD_HD + unit)] = h;
        }
        // (an odd number of tiles ends on the buffer that the next step begins with; the sums over h above end on the other one)
        if (MULTI && (pl.n_tiles & 1)) lds_barrier();
        b_before = b;
        b = b_next;
        b_next = next3(b);
    }
}

// ---------------------------------------------------------------- one row tile of the projection
__device__ __forceinline__ void seg_rows(const DevPtrs& d, const Words& x, const Pool& pl, int tile, int r, char* lds, Phases ps)
{
    const int wave = wave_id(), lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    float (*part)[NW][4][P_LD] = reinterpret_cast<float (*)[NW][4][P_LD]>(lds);  // [sixth of K][wave][element of the accumulator][lane]
    uint4 w[6];
#pragma unroll
    for (int kp = 0; kp < 6; ++kp) w[kp] = reinterpret_cast<const uint4*>(d.Wmel)[((size_t)r * NK_P + kp * NW + wave) * 64 + lane];
    const int rem = pl.rem[tile * 16 + col];
    // in the reduction: wave = four columns, thread = one of them and one of 16 rows
    const int my_col = (4 * wave + g) & 15, row16 = lane & 15, row = 16 * r + row16;
    const int el = row16 & 3, at = my_col + 16 * (row16 >> 2), m_off = (my_col * 16 + row16) * 4, m_buf = O_M + r * (SEG_SLOTS * 64);
    const int my_rem = wave < 4 && row < N_PROJ ? pl.rem[tile * 16 + my_col] : 0;
    const float bias = d.bmel[min(row, N_PROJ - 1)];
    auto product = [&](int kp, const uint4& b) __attribute__((always_inline)) {
        const floatx4 p = mfma_frag<h16_t>(w[kp], b, floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int i = 0; i < 4; ++i) part[kp][wave][i][lane] = p[i];
    };
    // a sixth's sum over the waves, rounded to 20 bits of mantissa as the step's kernels hand it over
    auto sixth = [&](int kp) __attribute__((always_inline)) {
        float v = kp == 0 ? bias : 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) v += part[kp][k][el][at];
        return __uint_as_float((__float_as_uint(v) + 8u) & ~15u);
    };
    int b = 0, b_next = 1;
    for (int s = 0; s < pl.n_steps; ++s) {
        const bool on = s < rem;
        uint4 ab[2], hd[4];
        bool ok = x.take<2, 64, 8>(O_A + b * B_A, wave, off_a(col, g), on, ab);
        if (s < my_rem) x.empty(m_off, m_buf + b_next * B_M);
        product(4, ab[0]);
        product(5, ab[1]);
        ps.sync(ok);
        const float v4 = sixth(4), v5 = sixth(5);
        if (ps.bad()) return give_up(d, pl, s);
        ok = x.take<4, B_FRAG>(O_HD + b * B_H, wave, off_hd(col, g), on, hd);
        stores_done();
#pragma unroll
        for (int kp = 0; kp < 4; ++kp) product(kp, hd[kp]);
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
__device__ __forceinline__ void seg_lead(const DevPtrs& d, const Words& x, const Pool& pl, int tile, char* lds, Phases ps)
{
    const int tid = threadIdx.x, wave = wave_id(), lane = tid & 63, col = lane & 15, g = lane >> 4;
    const int cur = pl.cur, n_steps = pl.n_steps, slot0 = tile * 16;
    uint16_t (*s_mel)[MEL_LD] = reinterpret_cast<uint16_t (*)[MEL_LD]>(lds);
    uint16_t (*s_hid)[HID_LD] = reinterpret_cast<uint16_t (*)[HID_LD]>(lds + 16 * MEL_LD * 2);
    constexpr int NK3 = MEL_ROWS / KB, NK4 = PRENET / KB;
    uint4 a3[2][NK3], a4[2][NK4];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int mt = 2 * wave + m;
#pragma unroll
        for (int f = 0; f < NK3; ++f) a3[m][f] = reinterpret_cast<const uint4*>(d.Wp1)[((size_t)mt * NK3 + f) * 64 + lane];
#pragma unroll
        for (int f = 0; f < NK4; ++f) a4[m][f] = reinterpret_cast<const uint4*>(d.Wp2)[((size_t)mt * NK4 + f) * 64 + lane];
    }
    const int rem = pl.rem[slot0 + col];
    // as a collector of the frame: thread = four rows of one slot
    constexpr int VEC = MEL_ROWS / 4;
    const int m_slot = min(tid / VEC, SEG_SLOTS - 1), m_row = tid % VEC * 4;
    const int m_rem = tid < SEG_SLOTS * VEC && m_row < N_PROJ ? pl.rem[slot0 + m_slot] : 0;
    const int m_t0 = d.n_steps[slot0 + m_slot] - m_rem, m_off = m_row / 16 * (SEG_SLOTS * 64) + m_slot * 64 + m_row % 16 * 4;     // [row tile][slot][16 rows]
    // the launches after this one read the half of this pair that belongs to their parity: it must not fall behind
    const int end_all = cur ^ (n_steps & 1);
    if (tile == 0 && tid == 0 && end_all != cur) d.wg_seq[end_all] = d.wg_seq[cur];
    int b = 0, b_next = 1;
    for (int s = 0; s < n_steps; ++s) {
        const bool on = s < rem, m_on = s < m_rem;
        if (on) x.empty4(off_hp(col, g), O_P + b_next * B_P + wave * B_FRAG);
        u32x4_t w = {0u, 0u, 0u, 0u};
        bool in = !m_on;
        for (int spin = 0; spin < x.polls && !in; ++spin) {
            Words::again();
            w = x.look4(m_off, O_M + b * B_M);
            in = m_row == N_MEL ? w.x != EMPTY : Words::full(w);
        }
        stores_done();
        if (m_row == N_MEL || !m_on) w.y = w.z = w.w = 0u;      // no rows beyond the stop row
        if (tid < SEG_SLOTS * VEC)
            *reinterpret_cast<uint2*>(&s_mel[m_slot][m_row]) = make_uint2(pack2<h16_t>(__uint_as_float(w.x), __uint_as_float(w.y)),
                                                                          pack2<h16_t>(__uint_as_float(w.z), __uint_as_float(w.w)));
        ps.sync(in);
        {
            uint4 bm[NK3];
#pragma unroll
            for (int f = 0; f < NK3; ++f) bm[f] = *reinterpret_cast<const uint4*>(&s_mel[col][f * KB + g * 8]);
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < NK3; ++f) acc = mfma_frag<h16_t>(a3[m][f], bm[f], acc);
                *reinterpret_cast<uint2*>(&s_hid[col][16 * (2 * wave + m) + 4 * g]) =
                    make_uint2(pack2<h16_t>(fmaxf(acc[0], 0.f), fmaxf(acc[1], 0.f)), pack2<h16_t>(fmaxf(acc[2], 0.f), fmaxf(acc[3], 0.f)));
            }
        }
        if (ps.bad()) return give_up(d, pl, s);
        lds_barrier();
        {
            uint4 bh[NK4];
#pragma unroll
            for (int f = 0; f < NK4; ++f) bh[f] = *reinterpret_cast<const uint4*>(&s_hid[col][f * KB + g * 8]);
            floatx4 acc[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int f = 0; f < NK4; ++f)
#pragma unroll
                for (int m = 0; m < 2; ++m) acc[m] = mfma_frag<h16_t>(a4[m][f], bh[f], acc[m]);
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int mt = 2 * wave + m;
                const unsigned lo = pack2<h16_t>(fmaxf(acc[m][0], 0.f), fmaxf(acc[m][1], 0.f)), hi = pack2<h16_t>(fmaxf(acc[m][2], 0.f), fmaxf(acc[m][3], 0.f));
                if (s + 1 < min(rem, n_steps)) {
                    x.put2(lo, hi, col * 64 + m * 32 + g * 8, O_P + b * B_P + wave * B_FRAG);
                } else if (on) {
                    h16_t* dst = reinterpret_cast<h16_t*>(d.xatt[cur ^ ((s + 1) & 1)]) + xoff<h16_t>(NK_A, slot0 + col, XA_P + 16 * mt + 4 * g);
                    *reinterpret_cast<uint2*>(dst) = make_uint2(lo, hi);
                }
            }
        }
        // the books, while the others go on
        if (m_on) {
            const size_t at = (size_t)(slot0 + m_slot) * d.max_steps + m_t0 + s;
            if (m_row < N_MEL) {
                *reinterpret_cast<u32x4_t*>(d.mel_ring + at * N_MEL + m_row) = w;
                *reinterpret_cast<u32x4_t*>(d.m_last + (slot0 + m_slot) * N_MEL + m_row) = w;
            } else {
                d.stop_ring[at] = __uint_as_float(w.x);
                // (no workgroup of this launch reads these two)
                d.t[slot0 + m_slot] = m_t0 + s + 1;
                if (s + 1 == m_rem) d.done[slot0 + m_slot] = 1;
            }
        }
        b = b_next;
        b_next = next3(b);
    }
}

// ---------------------------------------------------------------- one request's attention, shared by S workgroups
template <int S>
__device__ __forceinline__ void seg_lsa(const DevPtrs& d, const Words& x, const Pool& pl, int slot, int sp, char* lds, Phases ps)
{
    constexpr int FS = ENC / S, LPR = 64 / S, NA = 4 / S;                  // columns, lanes per row, position classes per lane
    const int cur = pl.cur, n_steps = pl.n_steps, in_tile = slot & 15;
    const int tid = threadIdx.x, wave = wave_id(), lane = tid & 63, jl = lane & 15, g = lane >> 4;
    float (*s_ctx)[ENC] = reinterpret_cast<float (*)[ENC]>(lds);
    float (*s_u)[U_PAD] = reinterpret_cast<float (*)[U_PAD]>(lds + NW * ENC * 4);
    float* s_e = reinterpret_cast<float*>(s_u + 2);
    float* s_q = s_e + MAX_ENC_LEN;
    float* s_v = s_q + ATT;
    float* s_red = s_v + ATT;
    float (*s_pair)[ATT] = reinterpret_cast<float (*)[ATT]>(s_red + 2 * NW);
    const int rem = __builtin_amdgcn_readfirstlane(pl.rem[slot]), L = __builtin_amdgcn_readfirstlane(d.L[slot]);
    if (rem == 0) return;
    const int steps = min(rem, n_steps), ntile = (L + 15) >> 4;
    const int ML = d.max_enc_len;
    const bf16_t* PMs = reinterpret_cast<const bf16_t*>(d.PM) + (size_t)slot * ML * ATT + 32 * g;
    LsaTile<h16_t> tile;
    {
        const uint4* kf = reinterpret_cast<const uint4*>(d.lsa_kfrag);
        const uint4* wf = reinterpret_cast<const uint4*>(d.lsa_wfrag);
#pragma unroll
        for (int i = 0; i < 4; ++i) tile.kA[i >> 1][i & 1] = kf[i * 64 + lane];
#pragma unroll
        for (int i = 0; i < 8; ++i) tile.wA[i] = wf[i * 64 + lane];
    }
    // the wave's rows of the processed memory stay in registers: of its tiles of positions up to 512 of them
    constexpr int NPM = S == 4 ? 1 : 2;
    u32x4_t pm0[NPM][4];
#pragma unroll
    for (int q = 0; q < NPM; ++q) {
        const bf16_t* pm = PMs + (size_t)min((sp + S * (wave + q * NW)) * 16 + jl, L - 1) * ATT;
#pragma unroll
        for (int i = 0; i < 4; ++i) pm0[q][i] = *reinterpret_cast<const u32x4_t*>(pm + 8 * i);
    }
    // and so do the rows of the memory (this workgroup's columns): NP passes of 32 positions
    constexpr int NP = S == 4 ? 16 : S == 2 ? 10 : 4;
    const int xw = wave * 4 + lane / LPR * NA;                             // this lane's first position class
    const bf16_t* Fslot = reinterpret_cast<const bf16_t*>(d.Fmem) + (size_t)slot * ML * ENC;
    const __amdgpu_buffer_rsrc_t f_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(Fslot), 0, L * ENC * 2, BUFFER_RSRC_RAW);
    const int f_col = (sp * FS + (lane % LPR) * 8) * 2;
    u32x4_t rows[NP][NA];
#pragma unroll
    for (int pp = 0; pp < NP; ++pp)
#pragma unroll
        for (int n = 0; n < NA; ++n) rows[pp][n] = __builtin_amdgcn_raw_buffer_load_b128(f_rsrc, (pp * 32 + xw + n) * ENC * 2 + f_col, 0, 0);
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

    // the energies of one workgroup's tiles lie together: [workgroup][its tiles][16 positions]
    const int e_slot = segment_energy_bytes(ML);
    auto e_off = [&](int j) { return (j >> 4) % S * (e_slot / S) + (j >> 4) / S * 64 + (j & 15) * 4; };
    // this thread's share of the query: four rows of two of its 32 partial products
    const int q_off = (tid >> 5) * 2 * ATT * 4 + (tid & 31) * 16, b_e = SEG_SLOTS * e_slot, e_at = O_E + in_tile * e_slot;
    const int k_a = sp * FS + tid, a_off = in_tile * (ENC * 2) + k_a * 2;
    int b = 0, b_next = 1;
    for (int s = 0; s < steps; ++s) {
#pragma unroll
        for (int i = 0; i < 4 * NPM; ++i) keep(pm0[i >> 2][i & 3]);
#pragma unroll
        for (int i = 0; i < NP * NA; ++i) keep(rows[i / NA][i % NA]);
        for (int tt = sp + S * wave; tt < ntile; tt += S * NW)
            if (g == 0 && tt * 16 + jl < L) x.empty(e_off(tt * 16 + jl), e_at + b_next * b_e);
        if (tid < FS && !(tid & 1)) x.empty(a_off, O_A + b_next * B_A);
        // the location features do not wait for the query
        uint4 bl0[NPM];
#pragma unroll
        for (int q = 0; q < NPM; ++q) bl0[q] = tile.loc(s_u[0], s_u[1], min((sp + S * (wave + q * NW)) * 16, (ntile - 1) * 16) + jl, g);
        {
            u32x4_t w0, w1;
            bool in = false;
            for (int spin = 0; spin < x.polls && !in; ++spin) {
                Words::again();
                w0 = x.look4(q_off, O_Q + b * B_Q + in_tile * B_QS);
                w1 = x.look4(q_off + ATT * 4, O_Q + b * B_Q + in_tile * B_QS);
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
        auto energies = [&](int tt, const uint4 (&pmc)[4], const uint4& bl) __attribute__((always_inline)) {
            const int j = tt * 16 + jl;
            float e = vsum;
#pragma unroll
            for (int at = 0; at < 8; ++at) {
                const floatx4 pl = mfma_frag<h16_t>(tile.wA[at], bl, *reinterpret_cast<const floatx4*>(&s_q[32 * g + 4 * at]));
                const float4 vv = *reinterpret_cast<const float4*>(&s_v[32 * g + 4 * at]);
                const uint4& u = pmc[at >> 1];
                const uint32_t w0 = (at & 1) ? u.z : u.x, w1 = (at & 1) ? u.w : u.y;
                e = fmaf(vv.x, half_one_minus_tanh(pl[0] + bf16_lo(w0)), e);
                e = fmaf(vv.y, half_one_minus_tanh(pl[1] + bf16_hi(w0)), e);
                e = fmaf(vv.z, half_one_minus_tanh(pl[2] + bf16_lo(w1)), e);
                e = fmaf(vv.w, half_one_minus_tanh(pl[3] + bf16_hi(w1)), e);
            }
            e += xor16(e);
            e += xor32(e);
            if (fast_softmax) e = __expf(e - bound);
            if (g == 0 && j < L) {
                s_e[j] = e;
                x.put(__float_as_uint(e), e_off(j), e_at + b * b_e);
            }
        };
#pragma unroll
        for (int q = 0; q < NPM; ++q) {
            const int tt = sp + S * (wave + q * NW);
            const uint4 pmc[4] = {as_uint4(pm0[q][0]), as_uint4(pm0[q][1]), as_uint4(pm0[q][2]), as_uint4(pm0[q][3])};
            if (tt < ntile) energies(tt, pmc, bl0[q]);
        }
        for (int tt = sp + S * (wave + NPM * NW); tt < ntile; tt += S * NW) {      // texts of more than 512 positions: from memory
            const bf16_t* pm = PMs + (size_t)min(tt * 16 + jl, L - 1) * ATT;
            uint4 pmc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) pmc[i] = *reinterpret_cast<const uint4*>(pm + 8 * i);
            energies(tt, pmc, tile.loc(s_u[0], s_u[1], tt * 16 + jl, g));
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
        auto add = [&](int n, int px, const uint4& r) __attribute__((always_inline)) {
            const float w = s_e[px];
            float fv[8];
            Vec16<bf16_t>::unpack(r, fv);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[n][i] = fmaf(w, fv[i], acc[n][i]);
        };
#pragma unroll
        for (int pp = 0; pp < NP; ++pp) {
            if (pp * 32 >= L) break;
#pragma unroll
            for (int n = 0; n < NA; ++n) add(n, pp * 32 + xw + n, as_uint4(rows[pp][n]));
        }
        for (int x0 = 32 * NP; x0 < L; x0 += 32 * 4 / NA) {                // longer texts: from memory
            uint4 more[4 / NA][NA];
#pragma unroll
            for (int pp = 0; pp < 4 / NA; ++pp)
#pragma unroll
                for (int n = 0; n < NA; ++n) more[pp][n] = buffer_load16(f_rsrc, (x0 + pp * 32 + xw + n) * ENC * 2 + f_col);
#pragma unroll
            for (int pp = 0; pp < 4 / NA; ++pp)
                if (x0 + pp * 32 < L)
#pragma unroll
                    for (int n = 0; n < NA; ++n) add(n, x0 + pp * 32 + xw + n, more[pp][n]);
        }
        // (classes held by one lane are paired here)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float t = acc[0][i];
            if constexpr (NA >= 2) t = acc[0][i] + acc[1][i];
            if constexpr (NA == 4) t = t + (acc[2][i] + acc[3][i]);
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
                float t = s_ctx[w][tid];
                if constexpr (S >= 2) t += s_ctx[w][LPR * 8 + tid];
                if constexpr (S == 4) t += s_ctx[w][2 * LPR * 8 + tid] + s_ctx[w][3 * LPR * 8 + tid];
                c += t;
            }
            const h16_t a = from_float<h16_t>(c * inv);
            const unsigned lo = a.bits, hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)lo, 0xB1, 0xf, 0xf, false);      // the neighbour's (lanes 1, 0, 3, 2)
            if (!(tid & 1)) x.put(lo | hi << 16, a_off, O_A + b * B_A);
            if (s + 1 == steps) {
                const int end = cur ^ (steps & 1);
                reinterpret_cast<h16_t*>(d.xatt[end])[xoff<h16_t>(NK_A, slot, XA_A + k_a)] = a;
                reinterpret_cast<h16_t*>(d.xdec[end ^ 1])[xoff<h16_t>(NK_D, slot, XD_A + k_a)] = a;
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

// Which workgroup does what.  Readers of the same words sit together, since an XCD's L2 takes a line that has been stored to from memory
// once for all of them: ATT and DEC fill XCDs 0 .. 3 in order, LSA and each tile's projection lie on 4 .. 7.  And at least eight CUs of every XCD
// stay free for work on other streams, whose launches are dealt over all XCDs: with XCDs filled to the last CU a vocoder beside the
// decoder waited for the end of a segment with each of its launches.  Against DEC and LSA on all XCDs: 1 request 9.9 -> 9.7 us a step,
// 16: 12.7 -> 11.2.  Faster but not taken: with all of ATT on one XCD and four or two LSA per request of two and three tiles, which leaves no CU of
// four XCDs free, 32 requests would take 13.4 us instead of 13.8, 48 of them 16.3 instead of 17.7.
constexpr int SEG_XCD_WGS = 24;                             // of ATT and DEC on an XCD; LSA, at most 16, and ROWS and LEAD fill the others as far
template <bool MULTI, int S>
__global__ __launch_bounds__(NT) void k_segment(DevPtrs d, int cur, int n_slots, int n_steps, char* words, char* words_next, int tile_bytes, int empty_bytes, SegmentLeft left)
{
    __shared__ __attribute__((aligned(16))) char lds[S_MAX];
    __shared__ int s_failed, s_rem[SEG_TILES * 16];
    const int n_tiles = (n_slots + 15) / 16;
    if (threadIdx.x == 0) s_failed = 0x7fffffff;
    if (threadIdx.x < SEG_TILES * 16) {
        const int sl = threadIdx.x;
        s_rem[sl] = sl < n_slots ? segment_left(d, left, sl) : 0;
    }
    for (int at = (blockIdx.x * NT + threadIdx.x) * 16; at < empty_bytes; at += gridDim.x * NT * 16)
        *reinterpret_cast<u32x4_t*>(words_next + at) = u32x4_t{EMPTY, EMPTY, EMPTY, EMPTY};
    __syncthreads();
    const Phases ps = {&s_failed};
    const Pool pl = {cur, n_steps, n_tiles, tile_bytes, s_rem};
    const Words x = {words, tile_bytes, d.wait_polls};
    const int xcd = blockIdx.x & 7, i = blockIdx.x >> 3;
    if (xcd < 4) {
        const int k = xcd * SEG_XCD_WGS + i;
        if (i >= SEG_XCD_WGS) return;
        if (k < 32) seg_att<MULTI>(d, x, pl, k, lds, ps);
        else seg_dec<MULTI>(d, x, pl, k - 32, lds, ps);
    } else if (i < 16) {
        const int slot = i / S * 4 + xcd - 4;
        if (slot < n_slots) seg_lsa<S>(d, x.of(slot >> 4, tile_bytes), pl, slot, i % S, lds, ps);
    } else if (xcd - 4 < n_tiles && i < 23) {
        const Words w = x.of(xcd - 4, tile_bytes);
        if (i < 22) seg_rows(d, w, pl, xcd - 4, i - 16, lds, ps);
        else seg_lead(d, w, pl, xcd - 4, lds, ps);
    }
}

}  // namespace

hipError_t launch_segment(const DevPtrs& d, int cur, int n_slots, int n_steps, int set, int empty_tiles, const SegmentLeft& left, hipStream_t s)
{
    const int n_tiles = (n_slots + 15) / 16;
    if (!d.seg_x || n_slots < 1 || n_slots > d.seg_slots || n_steps < 1 || (set & ~1) || empty_tiles < 0 || empty_tiles * SEG_SLOTS > d.seg_slots || d.stop_threshold >= 0.f)
        return hipErrorInvalidValue;
    const size_t tile_bytes = segment_tile_bytes(d.max_enc_len), set_bytes = d.seg_slots / SEG_SLOTS * tile_bytes;
    char* words = static_cast<char*>(d.seg_x);
    static_assert(4 * SEG_XCD_WGS == 32 + 64 && SEG_TILES <= 4, "ATT and DEC; a projection per XCD");
    static_assert(16 * 4 >= 4 * SEG_SLOTS && 16 * 4 >= 2 * 2 * SEG_SLOTS && 16 * 4 >= SEG_TILES * SEG_SLOTS, "LSA: four, two or one per slot");
#define SEG_ARGS dim3(8 * SEG_XCD_WGS), dim3(NT), 0, s, d, cur, n_slots, n_steps, words + set * set_bytes, words + (set ^ 1) * set_bytes, (int)tile_bytes, (int)(empty_tiles * tile_bytes), left
    if (n_tiles == 1) hipLaunchKernelGGL((k_segment<false, 4>), SEG_ARGS);
    else if (n_tiles == 2) hipLaunchKernelGGL((k_segment<true, 2>), SEG_ARGS);
    else hipLaunchKernelGGL((k_segment<true, 1>), SEG_ARGS);
#undef SEG_ARGS
    return hipGetLastError();
}

}  // namespace tts
