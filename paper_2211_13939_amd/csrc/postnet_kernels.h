// Host-visible launch wrapper of the PostNet kernels (postnet.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "stamps.h"

namespace tts {

constexpr int PN_LAYERS = 5;
constexpr int PN_TAPS = 5;
constexpr int PN_N_MEL = 80;
constexpr int PN_CIN0 = 96;          // the mel channels padded to whole 64-byte fragments in both dtypes
constexpr int PN_CHANNELS = 512;
constexpr int PN_COUT_LAST = 80;

// A call's stack of layers as one launch (conv5_chain.h): CHAIN_GROUPS groups of columns at most, each of one to three times
// chain_tiles column tiles (what 160 KB of LDS hold); CHAIN_LAYERS: most layers whose outputs the workgroups hand to each other.
constexpr int CHAIN_GROUPS = 8;
constexpr int CHAIN_LAYERS = 4;
constexpr int CHAIN_STATE_BYTES = 32;
constexpr int CHAIN_POLLS = 24;      // rounds of polls (0.8 us each) before a workgroup helps itself, the first time
constexpr int chain_tiles(size_t value_bytes) { return value_bytes == 2 ? 2 : 1; }
constexpr int chain_most_columns(size_t value_bytes) { return CHAIN_GROUPS * 3 * chain_tiles(value_bytes) * 16; }
constexpr int chain_column_bytes(size_t value_bytes) { return 16 * (int)value_bytes; }      // of one row tile's output
// column tiles a workgroup of a call: the fewest of one to three times chain_tiles that leave CHAIN_GROUPS groups at most
constexpr int chain_group_tiles(size_t value_bytes, int columns)
{
    const int unit = chain_tiles(value_bytes), tiles = (columns + 15) / 16;
    return tiles <= CHAIN_GROUPS * unit ? unit : tiles <= CHAIN_GROUPS * 2 * unit ? 2 * unit : 3 * unit;
}
// what a call stores: the columns of its groups, whole, of every layer
constexpr size_t chain_call_bytes(size_t value_bytes, int columns, int layers)
{
    const int group = chain_group_tiles(value_bytes, columns) * 16;
    return (size_t)((columns + group - 1) / group * group) * layers * PN_CHANNELS * value_bytes;
}
// One of the two sets of words, for calls of up to `columns` columns: those of the largest.  (A smaller call never stores more: a size of groups
// is left for the next one when eight of them are full.)
constexpr size_t chain_set_bytes(size_t value_bytes, long columns, int layers)
{
    const int most = chain_most_columns(value_bytes);
    return chain_call_bytes(value_bytes, columns < most ? (int)columns : most, layers);
}

struct PostnetPtrs {
    const void* W[PN_LAYERS];   // weight dtype, MFMA A-fragment order, k = tap * C_in(padded) + channel
    const float* b[PN_LAYERS];  // [c_out]
    void* act[2];               // activations between layers, fragment order, [column tile][channel fragment][lane][16 B]
    int* cmeta;                 // [columns padded to 16] (window length << 16) | index inside the window; 0 for padding
    int* orow;                  // [columns padded to 16] output row of the column, -1 = context or padding
    int n_mel;
    char* chain_words;          // calls that are one launch (conv5_chain.h): two sets of words, and the words that say which is in use;
    int* chain_state;           // null: no call is
    int chain_set_bytes;
    int wait_polls;             // ... and how often a workgroup polls for the others' words before it forms them itself
    Stamps stamps;
};

// Up to PN_META_WINDOWS windows of one call, as a kernel argument (no host-to-device copy): the device
// expands it into the per-column tables.
constexpr int PN_META_WINDOWS = 256;
struct PnWindows {
    int n;
    int col0[PN_META_WINDOWS];        // first column of the window
    int row0[PN_META_WINDOWS];        // output row of the window's first kept frame
    uint16_t len[PN_META_WINDOWS];    // frames in the window
    uint16_t keep[PN_META_WINDOWS];   // frames of context in front of the chunk
};
// The windows' tables and mel frames where the layers read them.  mel: device fp32 [n_col][n_mel]; n_col_pad: columns rounded up
// to whole tiles; `first`: the call's first windows (clears the padding columns too)
hipError_t launch_postnet_pack(const PostnetPtrs& d, int wdtype, const PnWindows& w, const float* mel, int n_col, int n_col_pad, bool first,
                               hipStream_t s);

// All of it as one launch: up to PN_META_WINDOWS windows of at most chain_most_columns columns
hipError_t launch_postnet_chain(const PostnetPtrs& d, int wdtype, const PnWindows& w, const float* mel, int n_col, float* out, hipStream_t s);

// The five layers behind launch_postnet_pack; out: device fp32 [kept rows][n_mel]
hipError_t launch_postnet(const PostnetPtrs& d, int wdtype, const float* mel, int n_col, float* out, hipStream_t s);

}  // namespace tts
