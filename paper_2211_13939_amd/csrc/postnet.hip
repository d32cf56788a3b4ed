// PostNet of the acoustic decoder on a ragged batch of windows (one window = the frames of one request's chunk plus the
// context in front of it): the per-column tables, the packing of the mel input and the five-layer stack.  The
// convolution kernels themselves are in conv5_kernels.h.
#include "conv5_kernels.h"

namespace tts {

// Everything the layers need of a call's windows, in one launch: the per-column tables from the window list, and the mel frames
// in the first layer's operand order, channels zero-padded to CIN.  A thread = 16 bytes of operand (8 or 4 channels of a column),
// one 16-byte store.  grid = (windows, pieces of 256 threads of the longest window); the call's first launch also clears the
// columns that pad the last tile.  Latency-bound at every size: 3.0 us for 3 windows, 3.4 us for 64, 4.0 us for 256.  As two
// launches with 2-byte stores a round of 64 windows took 86.8 us, like this 83.7 us; one of 3 windows 41.5 us, like this 38.3 us
// (two runs of one side differ by 3 %).
template <typename XT, int CIN>
__global__ __launch_bounds__(256) void k_pn_pack(PnWindows w, const float* __restrict__ mel, int n_col, int n_col_pad, int clear_pad,
                                                 XT* __restrict__ X, int* __restrict__ cmeta, int* __restrict__ orow)
{
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
}

hipError_t launch_postnet_pack(const PostnetPtrs& d, int wdtype, const PnWindows& w, const float* mel, int n_col, int n_col_pad, bool first,
                               hipStream_t s)
{
    int most = 0;
    for (int i = 0; i < w.n; ++i) most = w.len[i] > most ? w.len[i] : most;
    if (w.n < 1 || most < 1) return hipSuccess;
    auto go = [&](auto kern, int per_column, auto* x) {
        hipLaunchKernelGGL(kern, dim3(w.n, (most * per_column + 255) / 256), dim3(256), 0, s, w, mel, n_col, n_col_pad, first ? 1 : 0, x, d.cmeta, d.orow);
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
    hipError_t e = conv_layer<XT, C1, C, PN_EPI_TANH>(d.W[0], d.b[0], x0, x1, d.cmeta, n_ctiles, nullptr, 0, nullptr, nullptr, s);
    if (e == hipSuccess) e = conv_layer<XT, C, C, PN_EPI_TANH>(d.W[1], d.b[1], x1, x0, d.cmeta, n_ctiles, nullptr, 0, nullptr, nullptr, s);
    if (e == hipSuccess) e = conv_layer<XT, C, C, PN_EPI_TANH>(d.W[2], d.b[2], x0, x1, d.cmeta, n_ctiles, nullptr, 0, nullptr, nullptr, s);
    if (e == hipSuccess) e = conv_layer<XT, C, C, PN_EPI_TANH>(d.W[3], d.b[3], x1, x0, d.cmeta, n_ctiles, nullptr, 0, nullptr, nullptr, s);
    if (e == hipSuccess) e = conv_layer<XT, C, CO, PN_EPI_LAST>(d.W[4], d.b[4], x0, (XT*)nullptr, d.cmeta, n_ctiles, mel, d.n_mel, d.orow, out, s);
    return e;
}

hipError_t launch_postnet(const PostnetPtrs& d, int wdtype, const float* mel, int n_col, float* out, hipStream_t s)
{
    const int n_ctiles = (n_col + 15) / 16;
    if (n_ctiles < 1) return hipSuccess;
    return wdtype == 0 ? run_typed<float>(d, mel, n_ctiles, out, s) : run_typed<h16_t>(d, mel, n_ctiles, out, s);
}

}  // namespace tts
