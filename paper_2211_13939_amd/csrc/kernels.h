// Launch wrappers of the decoder-step kernels (definitions in kernels.hip).
#pragma once
#include "dev.h"

namespace tts {

// dtype codes as in the public header: 0 = fp32, 1 = bf16
struct StepLaunch {
    int wdtype;     // weights / activations
    int mdtype;     // encoder memory
    int n_blocks;   // the attention grid covers slots 0 .. n_blocks - 1 (all active slots lie below)
    int n_tiles;    // the projection grid covers 16-slot tiles 0 .. n_tiles - 1
    int lsa_split;  // workgroups per request in the attention kernel (1, 2 or 4; they split the context columns)
    int lstm_rows;  // row tiles per LSTM workgroup: 1 (all pool tiles each), 2 or 4 (1/2 or 1/4 of the pool tiles each)
    int proj_group; // workgroups per pool tile in the projection kernel: 6, 3 or 2 (fixed per pool; with pre_gates, n_tiles * proj_group <= 32)
    int att_lead;   // 1: the step begins with the attention LSTM's own launch (always, except in pools with d.p_x for a step
                    // whose predecessor in the same call formed it already); 0: it does not
    int att_tail;   // 1 (pools with d.p_x only): the step's last launch also forms the attention LSTM of the next step, which then
                    // has att_lead = 0.  The membership and the requests' states must not change between the two steps.
    int seg_steps;  // > 0: not one step but this many, as one launch (segment.hip): pools with d.seg_x and no stop threshold, n_blocks <= SEG_TILES * SEG_SLOTS,
                    // at least one running request takes each of the steps, the stream is not being captured (a replay would find the words
                    // of the replay before)
    int seg_set;    // which of the two sets of d.seg_x it uses: in turn, launch by launch
    int seg_empty;  // tiles of the other set it has to empty: those that the launch before used
    SegmentLeft seg_left; // by slot
    int pre_gates;  // 2: the projection's launch also forms the next step's gate pre-sums (d.pre_att / d.pre_dec; fp32: n_tiles <= PRESUM_SMALL_TILES),
                    // 1: the attention LSTM's only (pools of more than PRESUM_SMALL_TILES tiles: d.pre_dec is null);
                    // either way the attention LSTM hands the query to the attention kernel as rank-32 partial products (d.qpart)
};

// CUs the launches count on: the projection's launch of a pool with gate pre-sums has this many workgroups, one per CU,
// and the attention kernel at most this many
constexpr int MIN_DEVICE_CUS = 256;

// up to this many 16-slot tiles a pre-sum workgroup holds all its pool tiles' sums at once (both dtypes); beyond, it walks
// them with its row tiles' weights in registers (bf16 only)
constexpr int PRESUM_SMALL_TILES = 4;
// such a pool's attention LSTM writes this many partial products of the attention query per slot (d.qpart)
constexpr int QUERY_PARTIALS = 32;
// and its projection runs as this many workgroups per tile: d.proj_seq holds one sequence number for each, d.proj_part
// the 96 x 16 partial sums of all but the first (of all of them, and one more sequence number for the tile's leader, in
// the fused form of the last kernel: d.hdec_x)
constexpr int PROJ_GROUP = 6;       // the largest group
// d.seg_x: two sets, each for every pool tile three buffers of the words a segment's workgroups hand each other: h_att and h_dec
// (32 fragments of 1 KB), a (16), p (8), the query's partial products, the frame's rows and, per position of the longest text, the energies
constexpr size_t SEG_FIXED_BYTES = 3 * ((size_t)(32 + 32 + 16 + 8) * 1024 + (size_t)SEG_SLOTS * QUERY_PARTIALS * ATT * 4 + 96 * SEG_SLOTS * 4);
constexpr int segment_energy_bytes(int max_enc_len) { return (max_enc_len + 63) / 64 * 256; }      // per slot: a share for each of its workgroups
constexpr size_t segment_tile_bytes(int max_enc_len) { return SEG_FIXED_BYTES + (size_t)3 * SEG_SLOTS * segment_energy_bytes(max_enc_len); }
constexpr int segment_tiles(int max_pool) { return max_pool > SEG_TILES * SEG_SLOTS ? SEG_TILES : (max_pool + SEG_SLOTS - 1) / SEG_SLOTS; }
// fp32 weights and memory (segment32.hip), one tile: h_att and h_dec (64 fragments), a (32), p (16), the attention LSTM's pre-sums, and the rest
// as above
constexpr size_t SEG32_FIXED_BYTES =
    3 * ((size_t)(64 + 64 + 32 + 16 + HID / 4) * 1024 + (size_t)SEG_SLOTS * QUERY_PARTIALS * ATT * 4 + 96 * SEG_SLOTS * 4);
constexpr size_t segment32_bytes(int max_enc_len) { return SEG32_FIXED_BYTES + (size_t)3 * SEG_SLOTS * segment_energy_bytes(max_enc_len); }
constexpr size_t segment_bytes(int max_pool, int max_enc_len) { return 2 * segment_tiles(max_pool) * segment_tile_bytes(max_enc_len); }

// One decoder step (paper Eq. 2) for every request whose slot is flagged in d.live.
// `cur` selects which half of the double-buffered activations is read.
// If `ev` is given it holds N_STEP_KERNELS + 1 events: ev[0] is recorded before the
// first kernel and ev[i + 1] after kernel i (per-kernel device times).
// (Pools with d.hdec_x launch three kernels - the decoder LSTM is part of the last one - and record ev[3] right after ev[2].)
constexpr int N_STEP_KERNELS = 4;
hipError_t launch_segment(const DevPtrs& d, int cur, int n_slots, int n_steps, int set, int empty_tiles, const SegmentLeft& left, hipStream_t s);   // (launch_step's seg_steps)
hipError_t launch_segment32(const DevPtrs& d, int cur, int n_slots, int n_steps, int set, int empty_tiles, const SegmentLeft& left, hipStream_t s); // (fp32)
hipError_t launch_step(const DevPtrs& d, const StepLaunch& cfg, int cur, hipStream_t s, hipEvent_t* ev = nullptr);

hipError_t launch_set_live(const DevPtrs& d, const LiveArgs& args, hipStream_t s);
// chunks of `n` (<= MAX_POOL) requests from the mel ring to pinned host memory (its device address; 16-byte aligned)
hipError_t launch_stage_chunks(const DevPtrs& d, const StageArgs& sa, int n, int most_frames, float* dst, hipStream_t s);
// the whole per-slot state of `n` (<= MOVE_BATCH) running requests, each from its slot to a free one; the slots moved
// from and the slots moved to are disjoint
hipError_t launch_move_slots(const DevPtrs& d, int wdtype, int mdtype, const MoveArgs& mv, int n, hipStream_t s);
// `n` (<= JOIN_BATCH) requests join: state zeroed, F_enc (fp32, device) -> slot memory, processed memory PM = F W_mem^T
hipError_t launch_join(const DevPtrs& d, int wdtype, int mdtype, const JoinArgs& ja, int n, hipStream_t s);
// the gate pre-sums of one pool tile from activation half `nxt` (after a state overwrite between steps)
hipError_t launch_presum_tile(const DevPtrs& d, int wdtype, int tile, int nxt, hipStream_t s);
// p = Pre(m_last) into both activation buffers of one slot (after a state overwrite)
hipError_t launch_prenet_slot(const DevPtrs& d, int wdtype, int slot, hipStream_t s);

// one slot's piece [off, off+n) of a slot-tiled activation array with K elements per slot <-> fp32 device buffer
hipError_t launch_x_get(int wdtype, const void* X, int K, int slot, int off, int n, float* out, hipStream_t s);
hipError_t launch_x_set(int wdtype, void* X, int K, int slot, int off, int n, const float* in, hipStream_t s);

}  // namespace tts
