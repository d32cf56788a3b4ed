// A small call's stack of kernel-5 convolutions as ONE launch: the PostNet's five layers, and the encoder's three convolutions with the
// input projection behind them.
//
// As a launch per layer a small call is launches: each takes 5 to 8 us, of which the products are a fraction; the rest is its start, a trip
// for its weights, a trip for its columns.  Here a workgroup keeps its 16 rows and its columns (CT tiles of 16) from layer to layer: it has the
// next layer's weights on their way while it forms this one's sums, and takes the other workgroups' outputs as words (words.h) as they are
// stored.  The products, the eight partial sums and the order in which they meet are those of k_pn_conv, so are the results, bit for bit.
// What bounds it: a layer of three windows takes 2.8 us, 0.7 of them products (LDS reads), 0.5 their sums, tanh and stores, 1.6 until the others'
// words are in (one hop between compute units, 36 KB through one's L1); 3.2 us before the first layer's products, where the window list in
// the kernel's arguments lies in host memory.  Us a call, layer by layer -> as one launch, queued one behind the other (and, each waited for):
//   PostNet, windows of 50    1: 35.7 -> 23.6 (54 -> 35)   3: 36.6 -> 25.9 (56 -> 37)   8: 43.8 -> 33.2 (63 -> 45)   14: 46.7 -> 37.3
//            fp32             1: 47.2 -> 33.6 (65 -> 46)   3: 67.4 -> 49.0 (86 -> 61)   6: 88.6 -> 66.7 (107 -> 78)
//
// Words: [column group][layer][row tile] blocks, [column][16 channels] each: what one workgroup stores lies together, and a wave
// of its readers takes 1 KB of it with one load a lane.  There are two sets; a call uses the one whose turn it is and empties the other one.  Whose turn
// it is lies in device memory and changes with the call's last workgroup: a call that was captured goes on at every replay.
//
// Nobody has to be resident for the call to end.  A workgroup whose wait runs out (20 us; no call by itself keeps one waiting for 5) forms what it
// waits for: those that do so take the blocks of all layers in turn, from a counter, and form what is not there.  A block waits for blocks
// in front of it only, which others that run have taken or stored, so somebody always goes on; a block formed twice is stored twice with the same bits.
// So where the compute units are taken by other work, or by launches like this one on other streams that hold them while they wait, the
// workgroups that run go on alone, and the others find everything done.  And should one that has taken a block not get on with it (half a
// second), a workgroup that waits for it forms every block it needs by itself, layer by layer: then nothing is left to wait for.
#pragma once
#include "conv5_kernels.h"
#include "words.h"

namespace tts {

constexpr int CHAIN_RTS = PN_CHANNELS / 16;                // row tiles of an inner layer: workgroups per column group
constexpr int CHAIN_POLLS_THEN = 4;                        // CHAIN_POLLS, after the first time
constexpr int CHAIN_POLLS_LATE = 1 << 20;                  // ... for what others have taken, before it forms that too

template <typename XT, int CT_> struct ChainGeom {
    static constexpr int C = PN_CHANNELS, KB = Frag<XT>::KB, EPL = Frag<XT>::EPL;
    static constexpr int CT = CT_, COLS = CT * 16, ROWS = COLS + 2 * PN_HALO;
    static constexpr int PIECES = (int)sizeof(XT);                         // 16-byte pieces of 16 channels
    static constexpr int NKF = C / KB, NKT = PN_TAPS * NKF, NFW = NKT / PN_WAVES;
    // LDS: a plane per 16 bytes of channels, rows = columns, planes a multiple of 16 pieces apart (see ColGeom); row ROWS is zero
    static constexpr int PLANE = (ROWS + 1 + 15) / 16 * 16, X_BYTES = C * (int)sizeof(XT) * PLANE;
    static constexpr int SUBS = COLS * PIECES / 64, BLOCK = SUBS * 1024;   // a block is SUBS loads of a wave
    static constexpr int TAKES = CHAIN_RTS / PN_WAVES * SUBS;              // of them per wave and column group
    // the partial sums lie behind the columns, or, where LDS does not hold both, on top of them
    static constexpr int RED_BYTES = PN_WAVES * CT * 1024, LDS_MOST = 158 * 1024;
    static constexpr bool ON_TOP = X_BYTES + RED_BYTES > LDS_MOST;
    static constexpr int RED_AT = ON_TOP ? 0 : X_BYTES, LDS = ON_TOP ? X_BYTES : X_BYTES + RED_BYTES;
    static_assert(COLS * PIECES % 64 == 0 && BLOCK == COLS * chain_column_bytes(sizeof(XT)) && LDS <= LDS_MOST && RED_BYTES <= LDS, "whole loads");
    static_assert(NKT % PN_WAVES == 0 && 2 * PN_HALO * PIECES * CHAIN_RTS <= PN_THREADS, "whole fragments a wave, a halo piece a thread");
};

struct ChainArgs {
    const uint4* W[CHAIN_LAYERS];      // the layers whose outputs are words: A-fragment order, k = tap * C_in + channel
    const float* b[CHAIN_LAYERS];
    char* words;                       // two sets
    int set_bytes;
    int* state;                        // [0] which set is in use, [1] workgroups that are through, [2 + set] KB in use of it,
                                       // [4] blocks taken by workgroups that help themselves
    int groups;                        // column groups
    int polls;                         // CHAIN_POLLS or less (1: most take blocks from the counter; 0: nobody waits, every workgroup forms
                                       // what it needs by itself)
    Stamps stamps;                     // jobs that are a call of their own (TIMED)
};

// Where a wave's share of a row tile's weights lies: fragments first, first + step, ...  A fragment's place is a scalar offset, all loads share
// one address register; past the last fragment, and where there are none (count 0), they are zeros.
struct ChainWeights {
    __amdgpu_buffer_rsrc_t rsrc;
    int first, step;
    __device__ __forceinline__ ChainWeights(const uint4* W, int count, int rt, int first, int step)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(W + (size_t)rt * count * 64), 0, count * 1024, BUFFER_RSRC_RAW)), first(first), step(step) {}
    __device__ __forceinline__ uint4 at(int i) const
    {
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(threadIdx.x & 63) * 16, (first + i * step) * 1024, 0);
        return make_uint4(v.x, v.y, v.z, v.w);
    }
};

// piece (plane, row) of the columns in LDS
template <class G> __device__ __forceinline__ constexpr int chain_at(int plane, int row) { return (plane * G::PLANE + row) * 16; }

// the eight waves' partial sums of one row tile and CT column tiles: fragments wave, wave + 8, ... of k = (tap, channel fragment)
template <typename XT, class G, int NKF, int NFW, int NA, typename DONE>
__device__ __forceinline__ void chain_products(uint4 (&a)[NA], const unsigned char* s_x, const int (&tapmask)[G::CT], floatx4 (*red)[G::CT][64], DONE done)
{
    constexpr int NKT = PN_TAPS * NKF, CT = G::CT;
    static_assert(NFW <= NA, "room");
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4;
    int jl = lane & 15;
    asm volatile("" : "+v"(jl));               // the rows are made anew for every layer: kept from one to the next they cost more registers than the weights
    floatx4 acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
    constexpr int AHEAD = sizeof(XT) == 4 ? 1 : CT <= 2 ? 4 : 2;     // fragments between an operand's request and its use
    uint4 b[AHEAD][CT];
    auto request = [&](int i) __attribute__((always_inline)) {
        const int f = min(wave + i * PN_WAVES, NKT - 1);               // past the last fragment: any operand, the weights are zero
        const int tap = NKF % PN_WAVES == 0 ? i / (NKF < PN_WAVES ? 1 : NKF / PN_WAVES) : f / NKF, cf = f - tap * NKF;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int row = (tapmask[c] >> tap) & 1 ? c * 16 + jl + tap : G::ROWS;      // a tap that leaves its window meets zeros
            b[i % AHEAD][c] = *reinterpret_cast<const uint4*>(&s_x[chain_at<G>(cf * 4 + g, row)]);
        }
    };
#pragma unroll
    for (int i = 0; i < AHEAD && i < NFW; ++i) request(i);
#pragma unroll
    for (int i = 0; i < NFW; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        if (NKT % PN_WAVES == 0 || wave + i * PN_WAVES < NKT) {
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[c] = mfma_frag<XT>(a[i], b[i % AHEAD][c], acc[c]);
        }
        done(i);                               // fragment i's registers are free
        if (i + AHEAD < NFW) request(i + AHEAD);
    }
    if constexpr (G::ON_TOP) lds_barrier();
#pragma unroll
    for (int c = 0; c < CT; ++c) red[wave][c][lane] = acc[c];
}

// JOB: what is in front of the first layer and behind the last one
//   LAYERS  layers whose outputs are words; EPI: their activation; CIN: channels (padded) of the first one's input
//   windows what the thread knows of the call's windows, requested ahead of everything else
//   meta    columns col0 .. col0 + n: their place in their window, as in k_pn_conv (0: none), and what else last() wants to know of them
//   first   the first layer's input: columns col0 .. as rows of s_x (chain_at<G>)
//   goes_on whether a row tile's workgroups have a part in what follows the layers; HALO: whether that reads the columns on either side
//   weights LAST fragments for it; fetch: its bias, and four values more, requested ahead
//   last    what follows
// grid = column groups x CHAIN_RTS
template <typename XT, int CT, class JOB>
__global__ __launch_bounds__(PN_THREADS, 2) void k_conv_chain(JOB job, ChainArgs p)
{
    using G = ChainGeom<XT, CT>;
    constexpr int NKF0 = JOB::CIN / G::KB, NKT0 = PN_TAPS * NKF0, NFW0 = (NKT0 + PN_WAVES - 1) / PN_WAVES;
    constexpr int LAYERS = JOB::LAYERS;
    static_assert(LAYERS <= CHAIN_LAYERS && JOB::CIN <= G::C, "buffers");
    extern __shared__ __attribute__((aligned(16))) unsigned char s_x[];
    unsigned long long t0 = 0;
    if constexpr (JOB::TIMED) t0 = p.stamps.now();
    floatx4 (*red)[CT][64] = reinterpret_cast<floatx4 (*)[CT][64]>(s_x + G::RED_AT);
    __shared__ int s_meta[G::COLS], s_row[G::COLS], s_late, s_taken;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, jl = lane & 15, g = lane >> 4;
    const int my_rt = blockIdx.x % CHAIN_RTS, my_cg = blockIdx.x / CHAIN_RTS;
    const int set_bytes = p.set_bytes;
    const int turn = __builtin_amdgcn_readfirstlane(p.state[0]);
    const Words x = {p.words + (turn ? set_bytes : 0), set_bytes, p.polls};
    auto block = [&](int l, int cg, int rt) __attribute__((always_inline)) { return ((cg * LAYERS + l) * CHAIN_RTS + rt) * G::BLOCK; };

    int tapmask[CT];
    auto columns_of = [&](int cg, const auto& windows) __attribute__((always_inline)) {      // ends with all threads' s_meta in place
        job.meta(cg * G::COLS, G::COLS, windows, s_meta, s_row);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int m = s_meta[c * 16 + jl], t = m & 0xFFFF, T = m >> 16;
            int bits = 0;
#pragma unroll
            for (int d = -PN_HALO; d <= PN_HALO; ++d) bits |= (t + d >= 0 && t + d < T) ? (1 << (d + PN_HALO)) : 0;
            tapmask[c] = bits;
        }
    };
    auto zero_rows = [&]() __attribute__((always_inline)) {
        for (int i = tid; i < G::C * (int)sizeof(XT) / 16; i += PN_THREADS) *reinterpret_cast<uint4*>(&s_x[chain_at<G>(i, G::ROWS)]) = make_uint4(0, 0, 0, 0);
    };
    // a wave's share of a row tile's weights, of the layer at hand or of the one that follows
    constexpr int NA = JOB::LAST > G::NFW ? JOB::LAST : G::NFW;
    uint4 a[NA];
    auto bias_of = [&](const float* b, int rt) __attribute__((always_inline)) { return *reinterpret_cast<const floatx4*>(b + rt * 16 + 4 * g); };
    // the output of layer l of column group cg where the products read it; false: the wait ran out for some wave
    auto stage = [&](int l, int cg, bool halo, int polls) __attribute__((always_inline)) {
        const int hp = tid % G::PIECES, hc = tid / G::PIECES % (2 * PN_HALO), hrt = tid / (2 * PN_HALO * G::PIECES), hcg = hc < PN_HALO ? cg - 1 : cg + 1;
        const bool beside = halo && hrt < CHAIN_RTS && hcg >= 0 && hcg < p.groups;
        const int h_off = block(l, hcg, hrt) + ((hc < PN_HALO ? G::COLS - PN_HALO + hc : hc - PN_HALO) * G::PIECES + hp) * 16;
        u32x4_t w[G::TAKES], h = {0u, 0u, 0u, 0u};
        bool in = false;
        for (int spin = 0; spin < polls && !in; ++spin) {
            Words::again();
#pragma unroll
            for (int i = 0; i < G::TAKES; ++i) w[i] = x.look4(lane * 16, block(l, cg, wave + i / G::SUBS * PN_WAVES) + i % G::SUBS * 1024);
            if (beside) h = x.look4(h_off, 0);
            in = Words::full(h);
#pragma unroll
            for (int i = 0; i < G::TAKES; ++i) in = in && Words::full(w[i]);
        }
        if (!in) {
            s_late = 1;
        } else {
#pragma unroll
            for (int i = 0; i < G::TAKES; ++i)
                *reinterpret_cast<u32x4_t*>(&s_x[chain_at<G>((wave + i / G::SUBS * PN_WAVES) * G::PIECES + lane % G::PIECES, PN_HALO + (i % G::SUBS * 64 + lane) / G::PIECES)]) = w[i];
            if (halo && hrt < CHAIN_RTS)
                *reinterpret_cast<u32x4_t*>(&s_x[chain_at<G>(hrt * G::PIECES + hp, hc < PN_HALO ? hc : G::COLS + hc)]) = h;
        }
        lds_barrier();
        return s_late == 0;
    };
    // The caller's results may lie where his input lies.  They are written when every block of the first layer has been stored, so a workgroup that
    // finds its block stored by another one, after it has read the input, keeps its own to itself: it may be made of results.
    auto stored = [&](int cg, int rt) __attribute__((always_inline)) { return x.look(wave < CT ? (wave * 16 + jl) * G::PIECES * 16 + g * 4 * (int)sizeof(XT) : 0, block(0, cg, rt)); };
    // behind the products: the partial sums meet, and a layer's output goes out as words
    auto finish = [&](int l, int cg, int rt, const floatx4& bias, unsigned there) __attribute__((always_inline)) {
        lds_barrier();
        if (wave >= CT) return;
        floatx4 y = bias;
#pragma unroll
        for (int w = 0; w < PN_WAVES; ++w) y += red[w][wave][lane];
        const float y0 = pn_act<JOB::EPI>(y[0]), y1 = pn_act<JOB::EPI>(y[1]), y2 = pn_act<JOB::EPI>(y[2]), y3 = pn_act<JOB::EPI>(y[3]);
        const int at = (wave * 16 + jl) * G::PIECES * 16 + g * 4 * (int)sizeof(XT);
        if (there != EMPTY) return;
        if constexpr (sizeof(XT) == 2) x.put2(pack2<XT>(y0, y1), pack2<XT>(y2, y3), at, block(l, cg, rt));
        else x.put4(floatx4{y0, y1, y2, y3}, at, block(l, cg, rt));
    };
    // What layer l waits for and is not there, formed here: in few registers, which the layers need, and in its own time.  Blocks from the
    // counter (one taken is formed, whichever layer it is of); alone: all blocks in front of layer l, one behind the other, from the first
    // on, so that what a block is made of has been seen or stored by this workgroup
    auto help = [&](int l, bool alone) __attribute__((always_inline)) {
        int n_groups = p.groups;
        asm volatile("" : "+s"(n_groups));         // (none of this is made ahead of the layers)
        const int per_layer = n_groups * CHAIN_RTS;
#pragma unroll 1
        for (int j = -1; j + 1 < l * per_layer;) {
            if (tid == 0) s_taken = alone ? j + 1 : __hip_atomic_fetch_add(p.state + 4, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            j = s_taken;
            if (j >= LAYERS * per_layer) break;
            const int k = j / per_layer, cg = j / CHAIN_RTS % n_groups, rt = j % CHAIN_RTS, NKT = k == 0 ? NKT0 : G::NKT, NKF = NKT / PN_TAPS;
            Words::again();
            if (__syncthreads_and(wave >= G::SUBS || Words::full(x.look4(lane * 16, block(k, cg, rt) + wave * 1024)))) continue;
            columns_of(cg, job.windows());
            zero_rows();
            if (k == 0) job.template first<G>(cg * G::COLS - PN_HALO, s_x);
            else {
#pragma unroll 1
                for (int i = tid; i < G::ROWS * CHAIN_RTS * G::PIECES; i += PN_THREADS) {
                    const int plane = i / G::ROWS, row = i % G::ROWS, c = (cg * G::COLS - PN_HALO) + row;
                    u32x4_t v = {0u, 0u, 0u, 0u};
                    bool in = c < 0 || c >= n_groups * G::COLS;
#pragma unroll 1
                    for (int spin = 0; spin < CHAIN_POLLS_LATE && !in; ++spin) {
                        Words::again();
                        v = x.look4(block(k - 1, c / G::COLS, plane / G::PIECES) + (c % G::COLS * G::PIECES + plane % G::PIECES) * 16, 0);
                        in = Words::full(v);
                    }
                    if (!in) s_taken = -1;         // (never alone)
                    *reinterpret_cast<u32x4_t*>(&s_x[chain_at<G>(plane, row)]) = v;
                }
            }
            __syncthreads();
            if (s_taken < 0) break;
            const unsigned there = k == 0 ? stored(cg, rt) : EMPTY;
            const ChainWeights W(p.W[k], NKT, rt, wave, PN_WAVES);
            floatx4 acc[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int i = 0; wave + i * PN_WAVES < NKT; ++i) {
                const int f = wave + i * PN_WAVES, tap = f / NKF, cf = f - tap * NKF;
                const uint4 w = W.at(i);
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    acc[c] = mfma_frag<XT>(w, *reinterpret_cast<const uint4*>(&s_x[chain_at<G>(cf * 4 + g, (tapmask[c] >> tap) & 1 ? c * 16 + jl + tap : G::ROWS)]), acc[c]);
            }
            if constexpr (G::ON_TOP) lds_barrier();
#pragma unroll
            for (int c = 0; c < CT; ++c) red[wave][c][lane] = acc[c];
            finish(k, cg, rt, bias_of(p.b[k], rt), there);
            __syncthreads();
        }
        columns_of(my_cg, job.windows());
        if (tid == 0) s_late = 0;
        __syncthreads();
    };
    // A fragment of the next layer's weights is requested as soon as its predecessor's products are queued: while LDS and the matrix
    // pipes are busy and nobody polls.  (80 KB keep the unit's L1 busy for 0.5 us; requested behind the products they delay this layer's
    // words and the polls for the others'.)
    const ChainWeights W0(p.W[0], NKT0, my_rt, wave, PN_WAVES);
    auto weights_of = [&](int l) __attribute__((always_inline)) { return l < LAYERS ? ChainWeights(p.W[l], G::NKT, my_rt, wave, PN_WAVES) : job.weights(my_rt, wave); };
    floatx4 bias, with;
    {
        const auto windows = job.windows();
#pragma unroll
        for (int i = 0; i < NFW0; ++i) a[i] = W0.at(i);
        bias = bias_of(p.b[0], my_rt);
        if (tid == 0) s_late = 0;
        zero_rows();
        job.template first<G>(my_cg * G::COLS - PN_HALO, s_x);
        columns_of(my_cg, windows);
        const ChainWeights W1 = weights_of(1);
#pragma unroll
        for (int i = NFW0; i < NA; ++i) a[i] = i < G::NFW ? W1.at(i) : make_uint4(0, 0, 0, 0);
    }
    int polls = p.polls;
    auto take = [&](int l, bool halo) __attribute__((always_inline)) {
        if constexpr (G::ON_TOP) {
            lds_barrier();                         // the sums on top of the columns have been read
            zero_rows();
        }
        if (__builtin_expect(!stage(l - 1, my_cg, halo, polls), 0)) {
            bool in = false;
            if (p.polls > 0) {
                help(l, false);
                if (G::ON_TOP) zero_rows();
                in = stage(l - 1, my_cg, halo, CHAIN_POLLS_LATE);
            }
            if (!in) {
                help(l, true);
                if (G::ON_TOP) zero_rows();
                stage(l - 1, my_cg, halo, CHAIN_POLLS_LATE);
            }
            polls = min(polls, CHAIN_POLLS_THEN);
            const ChainWeights mine = weights_of(l);
#pragma unroll
            for (int i = 0; i < NA; ++i) a[i] = mine.at(i);
        }
    };
    {
        const ChainWeights W = weights_of(1);
        Words::again();
        const unsigned there = stored(my_cg, my_rt);
        chain_products<XT, G, NKF0, NFW0>(a, s_x, tapmask, red, [&](int i) __attribute__((always_inline)) { a[i] = W.at(i); });
        finish(0, my_cg, my_rt, bias, there);
    }
#pragma unroll 1
    for (int l = 1; l < LAYERS; ++l) {
        const ChainWeights W = weights_of(l + 1);
        bias = bias_of(p.b[l], my_rt);
        take(l, true);
        chain_products<XT, G, G::NKF, G::NFW>(a, s_x, tapmask, red, [&](int i) __attribute__((always_inline)) { a[i] = W.at(i); });
        finish(l, my_cg, my_rt, bias, EMPTY);
    }
    if (job.goes_on(my_rt)) {
        const ChainWeights W = weights_of(LAYERS);
#pragma unroll
        for (int i = G::NFW; i < NA; ++i) a[i] = W.at(i);
        job.template fetch<G>(my_cg * G::COLS, my_rt, s_row, bias, with);
        take(LAYERS, JOB::HALO);
        job.template last<G>(my_cg * G::COLS, my_rt, a, bias, with, s_x, red, tapmask, s_row);
    }
    // the other set, for the next call: what the call before used of it
    {
        const Words other = {p.words + (turn ? 0 : set_bytes), set_bytes, 0};
        const int n = __builtin_amdgcn_readfirstlane(p.state[2 + (turn ^ 1)]);
        for (int i = (int)blockIdx.x * PN_WAVES + wave; i < n; i += (int)gridDim.x * PN_WAVES) other.empty4(lane * 16, i * 1024);
    }
    __syncthreads();                       // every wave has read the state
    if (tid == 0) {
        const int through = __hip_atomic_fetch_add(p.state + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (through == (int)gridDim.x - 1) {
            p.state[0] = turn ^ 1;
            p.state[1] = 0;
            p.state[4] = 0;
            p.state[2 + turn] = p.groups * LAYERS * CHAIN_RTS * G::SUBS;
            p.state[2 + (turn ^ 1)] = 0;
        }
        if constexpr (JOB::TIMED) {
            p.stamps.begin(t0);
            p.stamps.end();
        }
    }
}

template <typename XT, int CT, class JOB>
inline hipError_t conv_chain_ct(const JOB& job, ChainArgs& p, int n_col, hipStream_t s)
{
    using G = ChainGeom<XT, CT>;
    auto kern = k_conv_chain<XT, CT, JOB>;
    static bool attr_set = false;                 // dynamic LDS above 64 KB has to be allowed once per kernel
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    p.groups = (n_col + G::COLS - 1) / G::COLS;
    if ((long)p.groups * JOB::LAYERS * CHAIN_RTS * G::BLOCK > p.set_bytes) return hipErrorInvalidValue;     // (made for smaller calls)
    hipLaunchKernelGGL(kern, dim3(p.groups * CHAIN_RTS), dim3(PN_THREADS), G::LDS, s, job, p);
    return hipGetLastError();
}
// Calls of up to MOST columns; CHAIN_GROUPS groups are a workgroup for every compute unit
template <typename XT, int MOST, class JOB>
inline hipError_t conv_chain(const JOB& job, ChainArgs& p, int n_col, hipStream_t s)
{
    constexpr int UNIT = chain_tiles(sizeof(XT));
    const int ct = chain_group_tiles(sizeof(XT), n_col);
    if (ct == UNIT) return conv_chain_ct<XT, UNIT>(job, p, n_col, s);
    if (ct == 2 * UNIT) return conv_chain_ct<XT, 2 * UNIT>(job, p, n_col, s);
    if constexpr (MOST > CHAIN_GROUPS * 2 * UNIT * 16) return conv_chain_ct<XT, 3 * UNIT>(job, p, n_col, s);
    return hipErrorInvalidValue;
}

}  // namespace tts
