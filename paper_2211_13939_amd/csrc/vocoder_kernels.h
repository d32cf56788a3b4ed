// Host-visible launch wrappers of the vocoder kernels (vocoder.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "stamps.h"

namespace tts {

constexpr int VOC_STAGES = 4;
constexpr int VOC_BLOCKS = 3;
constexpr int VOC_PAIRS = 3;
constexpr int VOC_N_MEL = 80;
constexpr int VOC_C0 = 128;
constexpr int VOC_HOP = 256;
constexpr int VOC_K_PRE = 7;
constexpr int VOC_K_POST = 7;
constexpr int VOC_MAX_BATCH = 256;
constexpr int VOC_MAX_OVERLAP = 16;
constexpr int voc_rate(int s) { return s < 2 ? 8 : 2; }
constexpr int voc_block_k(int b) { return b == 0 ? 3 : (b == 1 ? 7 : 11); }
constexpr int voc_dil(int p) { return 2 * p + 1; }
constexpr int voc_channels(int s) { return VOC_C0 >> (s + 1); }              // channels after stage s
// residual blocks of this many channels form pairs of positions: 2 C GEMM rows = (position of the pair, channel), k + 1 taps
constexpr bool voc_paired(int channels) { return channels <= 16; }
constexpr int voc_cum_rate(int s) { return s == 0 ? 8 : (s == 1 ? 64 : (s == 2 ? 128 : 256)); }   // positions per frame after stage s

constexpr int VOC_HAS_PREV = 2, VOC_LAST = 4;

// The smallest regions of the residual blocks with 64 channels: what a block's halo leaves of 128 positions comes out right, so a block with a
// shorter kernel has fewer regions.  A launch has a workgroup for every region that a window may have and no more, the longest kernel's first.  (With as many
// for every block, those without a region were every window's same ones, and an XCD gets every eighth workgroup: where a window has 8 or 16
// regions, of 8 or 16 frames, two XCDs had all of the shorter kernels'.  fp32, 40 windows of 8 frames / 20 of 16 / 6 of 32:
// 476 / 470 / 326 us a call, like this 392 / 384 / 248; two-byte, 1 / 4 of 48: 54.3 / 78.6 -> 54.1 / 76.8.)
constexpr int VOC_LEAST = 128;
constexpr int voc_least_out(int b) { return VOC_LEAST - 12 * (voc_block_k(b) - 1); }
struct VocLeast {
    int windows, n[VOC_BLOCKS];                                 // regions of a window
    __host__ __device__ int all() const { return windows * (n[0] + n[1] + n[2]); }
    // workgroup i's block, window and region
    __host__ __device__ int block(int i, int* window, int* tile) const
    {
        int b = VOC_BLOCKS - 1;
        for (; b > 0 && i >= windows * n[b]; --b) i -= windows * n[b];
        *window = i / n[b];
        *tile = i - *window * n[b];
        return b;
    }
};
inline VocLeast voc_least(int windows, int positions)
{
    VocLeast l{windows, {}};
    for (int b = 0; b < VOC_BLOCKS; ++b) l.n[b] = (positions + voc_least_out(b) - 1) / voc_least_out(b);
    return l;
}

struct VocoderPtrs {
    // weights in MFMA A-fragment order (weight dtype), k = tap * C_in + channel; biases fp32
    const void* pre_w;  const float* pre_b;
    const void* up_w[VOC_STAGES];  const float* up_b[VOC_STAGES];     // rows = phase * C_out + channel, taps = input offsets -1, 0, +1
    const void* res_w[VOC_STAGES][VOC_BLOCKS];      // a block's six convolutions one after the other, [2 pair + {0: dilated, 1: plain}]
    const float* res_b[VOC_STAGES][VOC_BLOCKS];     // [2 * VOC_PAIRS][channels]
    const void* post_w; const float* post_b;
    const float* alpha; const float* beta;    // [overlap * 256] fade-in / fade-out
    float* m_tail;      // [max_requests][overlap][n_mel]   tail(M_pre) of every state slot
    float* s_tail;      // [2][max_requests][overlap * 256] tail(S_pre): a slot's calls read one and write the other in turn
    size_t s_tail_turn; // elements between the two
    float* kept;        // [max_batch][overlap][n_mel]      last frames of this call's chunks, from its first launch to its last
    int* turn;          // [max_requests]  which of the two the slot's latest call writes (its calls' first launch changes it)
    int* len;           // [max_batch] frames in window i of this call (overlap frames in front included)
    int4* call;         // [max_batch] of window i: its frames, its first sample in the response, its state slot, the bits below and (bit 0) whose turn it is
    float* x0;          // [max_batch * window][c0]         conv_pre output
    float* y;           // upsampled activations of the current stage, [positions][channels]
    float* r[VOC_BLOCKS];   // output of every residual block of the current stage
    int overlap, window;    // window = overlap + max_chunk frames: the stride between windows, in frames
    Stamps stamps;
};

// The batch as a kernel argument (no host-to-device copy).
struct VocBatch {
    int n;
    int src_row[VOC_MAX_BATCH];      // first row of the chunk in d_mel
    int out_off[VOC_MAX_BATCH];      // first sample of the response in d_audio
    uint16_t n_frames[VOC_MAX_BATCH];
    uint16_t slot[VOC_MAX_BATCH];
    uint8_t has_prev[VOC_MAX_BATCH];
    uint8_t last[VOC_MAX_BATCH];
};

// One dynamic batch: splice [tail(M_pre), M_cur] (Eq. 3 line 1), G, fade of the heads against tail(S_pre) (Eq. 3 line 2), responses, both
// tails written back (Eq. 4)
hipError_t launch_vocoder(const VocoderPtrs& d, int wdtype, const VocBatch& b, const float* d_mel, float* d_audio, hipStream_t s);

}  // namespace tts
