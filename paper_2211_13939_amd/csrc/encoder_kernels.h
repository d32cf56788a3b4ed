// Host-visible launch wrapper of the encoder kernels (encoder.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "postnet_kernels.h"

namespace tts {

constexpr int ENC_TABLES = 4;
constexpr int ENC_CONVS = 3;
constexpr int ENC_DIM = 512;
constexpr int ENC_HID = 256;
constexpr int ENC_GATES = 4 * ENC_HID;      // gate rows per direction
constexpr int ENC_MAX_BATCH = 256;

// The three convolutions and the input projection, from the embedding in act[0] on, are one launch up to this many tokens.  Us a call, layer
// by layer -> as one launch, queued one behind the other (and, each waited for); two-byte: 1 request of 60 tokens 77.4 -> 71.6 (102 -> 91),
// 165: 150.2 -> 149.1 (176 -> 170), 384: 304.6 -> 299.8 (334 -> 325), 5 of 100: 116.3 -> 114.9 (145 -> 140), with six column tiles a
// workgroup, 7 of 100, 120.1 -> 122.9; fp32: 1 of 60 127.1 -> 120.1 (152 -> 140), 3 of 100 227.7 -> 210.2.
constexpr int enc_chain_columns(size_t value_bytes) { return value_bytes == 2 ? chain_most_columns(2) / 3 * 2 : chain_most_columns(4); }

struct EncoderPtrs {
    const float* tables[ENC_TABLES];        // fp32 [vocab][dim]
    const void* conv_w[ENC_CONVS];          // weight dtype, A-fragment order, k = tap * dim + channel
    const float* conv_b[ENC_CONVS];
    const void* w_ih[2];                    // weight dtype, A-fragment order, rows permuted to unit-major / gate-minor
    const void* w_hh[2];
    const float* b[2];                      // permuted like the rows
    void* act[2];                           // activations of the convolution stack, fragment order
    int* cmeta;                             // per column: (request length << 16) | position inside the request
    uint32_t* hx;                           // fp32: [2][requests][2][ENC_HID] words through which workgroups exchange h
    float* xproj;                           // [2][max_tokens][ENC_GATES]: W_ih x + b of every token, both directions
    char* chain_words;                      // calls whose convolutions are one launch: as in PostnetPtrs
    int* chain_state;
    int chain_set_bytes;
    int max_tokens;
    int n_cu;                               // compute units of the device
    int wait_polls;                         // how often a workgroup polls a partner's word before it gives up
    int* gave_up;                           // fp32: device word, raised by a workgroup that gave up
};

// what a call hands over through pinned host memory (device addresses), one entry per token
struct EncStaged {
    const int4* ids;                        // the ids of the four tables
    const int* meta;                        // (request length << 16) | position inside the request
};

// w lists the requests (PnWindows: col0 = first token, len); out fp32 [n_col][2 hid]
hipError_t launch_encoder(const EncoderPtrs& d, int wdtype, const PnWindows& w, int n_col, const EncStaged& staged, float* out, hipStream_t s);

}  // namespace tts
