// PostNet of the acoustic decoder on a ragged batch of windows (one window = the frames of one request's chunk plus the
// context in front of it): the per-column tables, the packing of the mel input and the five-layer stack.  The
// convolution kernels themselves are in conv5_kernels.h.
#include "conv5_chain.h"

namespace tts {

// Everything the layers need of a call's windows, in one launch: the per-column tables from the window list, and the mel frames
// in the first layer's operand order, channels zero-padded to CIN.  A thread = 16 bytes of operand (8 or 4 channels of a column),
// one 16-byte store.  grid = (windows, pieces of 256 threads of the longest window); the call's first launch also clears the
// columns that pad the last tile.  Latency-bound at every size: 3.0 us for 3 windows, 3.4 us for 64, 4.0 us for 256.  As two
// launches with 2-byte stores a round of 64 windows took 86.8 us, like this 83.7 us; one of 3 windows 41.5 us, like this 38.3 us
// (two runs of one side differ by 3 %).
template <typename XT, int CIN>
__global__ __launch_bounds__(256) void k_pn_pack(PnWindows w, const float* __restrict__ mel, int n_col, int n_col_pad, int clear_pad,
                                                 XT* __restrict__ X, int* __restrict__ cmeta, int* __restrict__ orow, Stamps stamps)
{
    const unsigned long long t0 = stamps.now();
    constexpr int KB = Frag<XT>::KB, EPL = Frag<XT>::EPL, NG = CIN / EPL;
    static_assert(PN_N_MEL % EPL == 0 && CIN % EPL == 0, "a piece is all mel channels or all padding");
    const int i = blockIdx.x, first = blockIdx.y * 256 + threadIdx.x;
    const int T = w.len[i], keep = w.keep[i], col0 = w.col0[i], row0 = w.row0[i];
    for (int e = first; e < T * NG; e += gridDim.y * 256) {
        const int t = e / NG, ch = (e - t * NG) * EPL, col = col0 + t;
        float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (ch < PN_N_MEL) {
#pragma unroll
            for (int k = 0; k < EPL; k += 4) {
                const float4 m = *reinterpret_cast<const float4*>(mel + (size_t)col * PN_N_MEL + ch + k);
                v[k] = m.x; v[k + 1] = m.y; v[k + 2] = m.z; v[k + 3] = m.w;
            }
        }
        XT* dst = X + xoff<XT>(CIN / KB, col, ch);
        if constexpr (sizeof(XT) == 2) *reinterpret_cast<uint4*>(dst) = make_uint4(pack2<XT>(v[0], v[1]), pack2<XT>(v[2], v[3]), pack2<XT>(v[4], v[5]), pack2<XT>(v[6], v[7]));
        else *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
        if (ch == 0) {
            cmeta[col] = (T << 16) | t;
            orow[col] = t >= keep ? row0 + (t - keep) : -1;
        }
    }
    if (clear_pad && i == 0)
        for (int e = first; e < (n_col_pad - n_col) * NG; e += gridDim.y * 256) {
            const int c = e / NG, ch = (e - c * NG) * EPL, col = n_col + c;
            *reinterpret_cast<uint4*>(X + xoff<XT>(CIN / KB, col, ch)) = make_uint4(0, 0, 0, 0);
            if (ch == 0) {
                cmeta[col] = 0;
                orow[col] = -1;
            }
        }
    if (clear_pad) stamps.begin(t0);
}

hipError_t launch_postnet_pack(const PostnetPtrs& d, int wdtype, const PnWindows& w, const float* mel, int n_col, int n_col_pad, bool first,
                               hipStream_t s)
{
    int most = 0;
    for (int i = 0; i < w.n; ++i) most = w.len[i] > most ? w.len[i] : most;
    if (w.n < 1 || most < 1) return hipSuccess;
    auto go = [&](auto kern, int per_column, auto* x) {
        hipLaunchKernelGGL(kern, dim3(w.n, (most * per_column + 255) / 256), dim3(256), 0, s, w, mel, n_col, n_col_pad, first ? 1 : 0, x, d.cmeta, d.orow, d.stamps);
    };
    if (wdtype == 0) go(k_pn_pack<float, PN_CIN0>, PN_CIN0 / Frag<float>::EPL, reinterpret_cast<float*>(d.act[0]));
    else go(k_pn_pack<h16_t, PN_CIN0>, PN_CIN0 / Frag<h16_t>::EPL, reinterpret_cast<h16_t*>(d.act[0]));
    return hipGetLastError();
}

template <typename XT>
static hipError_t run_typed(const PostnetPtrs& d, const float* mel, int n_ctiles, float* out, hipStream_t s)
{
    constexpr int C1 = PN_CIN0, C = PN_CHANNELS, CO = PN_COUT_LAST;
    XT* x0 = reinterpret_cast<XT*>(d.act[0]);
    XT* x1 = reinterpret_cast<XT*>(d.act[1]);
    hipError_t e = conv_layer<XT, C1, C, PN_EPI_TANH>(d.W[0], d.b[0], x0, x1, d.cmeta, n_ctiles, nullptr, 0, nullptr, nullptr, Stamps{}, s);
    if (e == hipSuccess) e = conv_layer<XT, C, C, PN_EPI_TANH>(d.W[1], d.b[1], x1, x0, d.cmeta, n_ctiles, nullptr, 0, nullptr, nullptr, Stamps{}, s);
    if (e == hipSuccess) e = conv_layer<XT, C, C, PN_EPI_TANH>(d.W[2], d.b[2], x0, x1, d.cmeta, n_ctiles, nullptr, 0, nullptr, nullptr, Stamps{}, s);
    if (e == hipSuccess) e = conv_layer<XT, C, C, PN_EPI_TANH>(d.W[3], d.b[3], x1, x0, d.cmeta, n_ctiles, nullptr, 0, nullptr, nullptr, Stamps{}, s);
    if (e == hipSuccess) e = conv_layer<XT, C, CO, PN_EPI_LAST>(d.W[4], d.b[4], x0, (XT*)nullptr, d.cmeta, n_ctiles, mel, d.n_mel, d.orow, out, d.stamps, s);
    return e;
}

// The whole call as one launch (conv5_chain.h): the first layer reads the caller's frames, four layers' outputs are words, the last one
// (five row tiles: the workgroups of the others are done before it) writes the chunks' own frames.
template <typename XT> struct PnChain {
    static constexpr bool TIMED = true;
    static constexpr int LAYERS = PN_LAYERS - 1, CIN = PN_CIN0, EPI = PN_EPI_TANH, EPL = Frag<XT>::EPL;
    static constexpr int LAST = PN_TAPS * PN_CHANNELS / Frag<XT>::KB / PN_WAVES;
    PnWindows w;
    const float* mel;
    int n_col;
    const uint4* W;
    const float* b;
    float* out;
    __device__ __forceinline__ int4 windows() const                        // a thread = a window (a kernel argument lies in host memory: 1.8 us)
    {
        const int k = threadIdx.x;
        return k < w.n ? make_int4(w.col0[k], w.row0[k], w.len[k], w.keep[k]) : make_int4(0, 0, 0, 0);
    }
    __device__ __forceinline__ void meta(int col0, int n, const int4& win, int* s_meta, int* s_row) const
    {
        if ((int)threadIdx.x < n) {
            s_meta[threadIdx.x] = 0;
            s_row[threadIdx.x] = -1;
        }
        __syncthreads();
        const int first = win.x, T = win.z, keep = win.w, end = min(first + T, col0 + n);
        for (int c = max(first, col0); c < end; ++c) {
            s_meta[c - col0] = (T << 16) | (c - first);
            s_row[c - col0] = c - first >= keep ? win.y + (c - first - keep) : -1;
        }
    }
    template <class G> __device__ __forceinline__ void first(int col0, unsigned char* s_x) const
    {
        constexpr int NP = CIN / EPL;
        for (int p = threadIdx.x; p < G::ROWS * NP; p += PN_THREADS) {
            const int row = p / NP, ch = (p - row * NP) * EPL, col = col0 + row;
            float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (col >= 0 && col < n_col && ch < PN_N_MEL) {
#pragma unroll
                for (int k = 0; k < EPL; k += 4) {
                    const float4 m = *reinterpret_cast<const float4*>(mel + (size_t)col * PN_N_MEL + ch + k);
                    v[k] = m.x; v[k + 1] = m.y; v[k + 2] = m.z; v[k + 3] = m.w;
                }
            }
            unsigned char* dst = &s_x[chain_at<G>(p - row * NP, row)];
            if constexpr (sizeof(XT) == 2) *reinterpret_cast<uint4*>(dst) = make_uint4(pack2<XT>(v[0], v[1]), pack2<XT>(v[2], v[3]), pack2<XT>(v[4], v[5]), pack2<XT>(v[6], v[7]));
            else *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
    static constexpr bool HALO = true;
    __device__ __forceinline__ bool goes_on(int rt) const { return rt < PN_COUT_LAST / 16; }
    __device__ __forceinline__ ChainWeights weights(int rt, int wave) const
    {
        return goes_on(rt) ? ChainWeights(W, LAST * PN_WAVES, rt, wave, PN_WAVES) : ChainWeights(W, 0, 0, 0, 0);
    }
    template <class G>
    __device__ __forceinline__ void fetch(int col0, int rt, const int* s_row, floatx4& bias, floatx4& with) const
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
        const int ch = rt * 16 + 4 * (lane >> 4), col = wave * 16 + (lane & 15);
        if (!goes_on(rt) || wave >= G::CT) return;
        bias = *reinterpret_cast<const floatx4*>(b + ch);
        if (s_row[col] >= 0) with = *reinterpret_cast<const floatx4*>(mel + (size_t)(col0 + col) * PN_N_MEL + ch);
    }
    template <class G, int NA>
    __device__ __forceinline__ void last(int col0, int rt, uint4 (&a)[NA], const floatx4& bias, const floatx4& with, const unsigned char* s_x, floatx4 (*red)[G::CT][64],
                                         const int (&tapmask)[G::CT], const int* s_row) const
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, ch = rt * 16 + 4 * (lane >> 4);
        chain_products<XT, G, G::NKF, G::NFW>(a, s_x, tapmask, red, [](int) {});
        lds_barrier();
        const int row = wave < G::CT ? s_row[wave * 16 + (lane & 15)] : -1;
        if (row < 0) return;
        floatx4 y = bias;
#pragma unroll
        for (int w8 = 0; w8 < PN_WAVES; ++w8) y += red[w8][wave][lane];
        *reinterpret_cast<float4*>(out + (size_t)row * PN_N_MEL + ch) = make_float4(with[0] + y[0], with[1] + y[1], with[2] + y[2], with[3] + y[3]);
    }
};

hipError_t launch_postnet_chain(const PostnetPtrs& d, int wdtype, const PnWindows& w, const float* mel, int n_col, float* out, hipStream_t s)
{
    if (w.n < 1 || n_col < 1) return hipSuccess;
    ChainArgs p{};
    for (int l = 0; l < PN_LAYERS - 1; ++l) {
        p.W[l] = (const uint4*)d.W[l];
        p.b[l] = d.b[l];
    }
    p.words = d.chain_words;
    p.state = d.chain_state;
    p.set_bytes = d.chain_set_bytes;
    p.polls = d.wait_polls < CHAIN_POLLS ? d.wait_polls : CHAIN_POLLS;
    p.stamps = d.stamps;
    auto go = [&](auto job, auto type) {
        job.w = w;
        job.mel = mel;
        job.n_col = n_col;
        job.W = (const uint4*)d.W[PN_LAYERS - 1];
        job.b = d.b[PN_LAYERS - 1];
        job.out = out;
        return conv_chain<decltype(type), chain_most_columns(sizeof(type))>(job, p, n_col, s);
    };
    return wdtype == 0 ? go(PnChain<float>{}, float{}) : go(PnChain<h16_t>{}, h16_t{});
}

hipError_t launch_postnet(const PostnetPtrs& d, int wdtype, const float* mel, int n_col, float* out, hipStream_t s)
{
    const int n_ctiles = (n_col + 15) / 16;
    if (n_ctiles < 1) return hipSuccess;
    return wdtype == 0 ? run_typed<float>(d, mel, n_ctiles, out, s) : run_typed<h16_t>(d, mel, n_ctiles, out, s);
}

}  // namespace tts
