// Launch plan and workspace layout shared by the C-ABI host code and the
// gfx950 kernels of the ASD verifier.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace asd {

// Threads per workgroup of the row kernel: four 64-wide wavefronts.
constexpr int kRowThreads = 256;
// Threads of the per-request scan kernel.
constexpr int kScanThreads = 256;
// Largest number of vocabulary splits of one row.
constexpr int kMaxSplits = 64;

// One tile's best candidate when a row is split over several workgroups:
// (key, column) packed so that a larger value means a greater logit and, among
// equal logits, a lower column; the logit's binary32 bit pattern; and, in the
// tile that owns the draft token's column, that column's logit.
struct alignas(16) TilePartial {
    unsigned long long packed;
    uint32_t bits;
    uint32_t draft_bits;
};

// Per-row result consumed by the per-request scan: argmax in the low 30 bits,
// bit 31 = mismatch (draft != argmax), bit 30 = draft id outside [0, V);
// and the regret r = fl32(z(y*) - z(x)).
struct alignas(8) RowRecord {
    uint32_t y_flags;
    float regret;
};

// Bits of the sticky per-device error word (the values of ASD_DEVERR_*).
constexpr uint32_t kErrNegativeK = 1u;   // a request with K < 0, read as K = 0
constexpr uint32_t kErrRows = 2u;        // a request whose rows lie outside the batch
constexpr uint32_t kErrCommit = 4u;      // a verified request whose tokens were not committed

// Address of this device's error word (device memory, 4 bytes), valid on the
// device current at the call.
hipError_t error_word_address(uint32_t** ptr);

// Size of the fixed per-device workspace of asd_verify_static (the value of
// ASD_STATIC_SCRATCH_BYTES).
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;

// Device address of that workspace on the device current at the call, looked
// up once per device and cached.
hipError_t static_scratch_address(void** ptr);

constexpr uint32_t kMismatchBit = 0x80000000u;
constexpr uint32_t kBadDraftBit = 0x40000000u;
constexpr uint32_t kArgmaxMask = 0x3fffffffu;

struct Plan {
    int elem_bytes;          // 2 (bf16) or 4 (f32)
    int64_t vocab;
    int64_t rows;
    int32_t num_requests;
    int splits;              // S >= 1 vocabulary splits per row
    int64_t chunk_vecs;      // 16-byte vectors per split (multiple of kRowThreads)
    // Workspace layout (byte offsets from the workspace base; 256-byte aligned).
    // Nothing in it is carried from one call to the next.
    size_t off_offsets;      // int64 [num_requests]: packed row offsets
    size_t off_records;      // RowRecord [rows] (splits == 1)
    size_t off_partials;     // TilePartial [rows * splits] (splits > 1)
    size_t ws_bytes;
};

// Arguments of one verifier call after host validation.
struct CallArgs {
    const void* logits = nullptr;
    int32_t num_requests = 0;
    const int32_t* draft_tokens = nullptr;
    const int32_t* block_lens = nullptr;
    const int64_t* row_offsets = nullptr;
    const float* tau = nullptr;
    const int32_t* exc_cap = nullptr;
    float2* budget = nullptr;          // (B, s) per request
    int32_t* out_accept_len = nullptr;
    int32_t* out_next_token = nullptr;
    int32_t* out_argmax = nullptr;
    float* out_regret = nullptr;
    bool raw_gate = false;             // gate on r <= g instead of r / q <= g
    // Commit in the same pass (asd_verify_commit); tokens == nullptr: none.
    int32_t* commit_tokens = nullptr;  // [num_requests][commit_capacity]
    int64_t commit_capacity = 0;
    int64_t* commit_seq_len = nullptr; // [num_requests], advanced in place
    int32_t* commit_done = nullptr;    // [num_requests] or nullptr
};

Plan make_plan(int elem_bytes, int64_t vocab, int64_t rows, int32_t num_requests,
               int num_cus);

// Plans small enough for one launch (row pass and scan in one kernel; see
// asd_row_scan_kernel): few tiles, and few requests, since the last tile scans
// every request with its four wavefronts.  A second launch costs the host 2.8 us;
// counting on one counter costs each tile a wait for its output and about 10 ns.
// The limit lies where calls of the Python binding cross, which the host bounds
// when they take two launches.  us a call, one launch against two, one box:
//
//   tiles               63 (9 rows of 32,000 f32)   91     96     104    120
//   Python, in a row    7.3 / 8.5      7.6-8.1 / 8.4   8.0 / 8.4   8.0 / 8.4   8.5 / 8.4
//   C, in a row         7.3 / 6.4      7.6-8.0 / 6.6   8.0 / 6.5   7.9 / 6.8   8.4 / 6.7
//   one call alone      19.8 / 19.0    20.2 / 19.4     20.4 / 19.4   20.4 / 19.7   20.9 / 19.7
//   host of the call    5.8 / 8.7
//
// (The Python figures are of the public functions; C stands for the entry point
// called through the binding's native function.)  Single launches of more tiles
// lose everywhere: 270 tiles 11.3 / 8.1 us, 720 tiles 20.1 / 10.4.
constexpr int64_t kSingleLaunchMaxTiles = 96;
constexpr int32_t kSingleLaunchMaxRequests = 8;   // two per wavefront of the last tile
inline bool single_launch(const Plan& p) {
    return p.rows * p.splits <= kSingleLaunchMaxTiles &&
           p.num_requests <= kSingleLaunchMaxRequests;
}

// Bytes of the header in front of every library-owned workspace (and of the
// fixed scratch): the counter of single-launch calls, zero between calls.
constexpr size_t kCounterHeaderBytes = 256;

// `counter`: a zero counter the call may use for the single-launch form (it
// leaves it zero), or nullptr for the two-kernel form.
hipError_t launch_verify(const Plan& plan, const CallArgs& args, void* workspace,
                         unsigned* counter, hipStream_t stream);

// The row pass of `plan` alone: the row kernel on the plan's tile grid, every
// tile writing its TilePartial at out_partials[row * splits + split].
hipError_t launch_row_pass(const Plan& plan, const void* logits, const int32_t* draft_tokens,
                          void* out_partials, hipStream_t stream);

// One vocabulary shard: rows of `shard_vocab` columns that are columns
// [vocab_offset, vocab_offset + shard_vocab) of the full vocabulary.  Writes one
// TilePartial per row.
hipError_t launch_shard_argmax(int elem_bytes, const void* shard_logits, int64_t shard_vocab,
                               int64_t vocab_offset, int64_t rows, const int32_t* draft_tokens,
                               void* out_partials, hipStream_t stream);

// Combine the partials of `num_shards` shards ([shard][row], shard k holding
// columns [k shard_vocab, (k + 1) shard_vocab)) and run Algorithm 1.
// `packed_offsets` (int64 [num_requests]) is scratch for the packed layout; when
// it is NULL too, each scan wavefront sums its request's offset itself (meant
// for at most kWaveOffsetsMaxRequests requests).
constexpr int32_t kWaveOffsetsMaxRequests = 1024;
hipError_t launch_verify_partials(const void* partials, int num_shards, int64_t shard_vocab,
                                  int64_t vocab, int64_t rows, const CallArgs& args,
                                  int64_t* packed_offsets, hipStream_t stream);

// Opportunity statistic (Eq. 4): at most this many (tau, p) pairs per call.
constexpr int kMaxOpportunityPairs = 1024;

hipError_t launch_opportunity(const int32_t* draft_tokens, const int32_t* row_argmax,
                              const float* row_regret, int64_t vocab, int32_t num_requests,
                              int64_t total_rows, const int32_t* block_lens,
                              const int64_t* row_offsets, const float* taus, int32_t num_taus,
                              const int32_t* ps, int32_t num_ps, unsigned long long* counts,
                              unsigned long long* mismatches, hipStream_t stream);

hipError_t launch_commit(const int32_t* draft_tokens, const int32_t* block_lens,
                         const int64_t* row_offsets, int32_t num_requests, int64_t total_rows,
                         const int32_t* accept_len, const int32_t* next_token, int32_t* tokens,
                         int64_t capacity, int64_t* seq_len, int32_t* committed,
                         hipStream_t stream);

// LM-head-fused verification: workspace = uint64 best [rows], uint32 draft
// logits [rows] at lmhead_draft_offset(rows), int64 packed offsets
// [num_requests] at lmhead_offsets_offset(rows).
inline size_t lmhead_draft_offset(int64_t rows) {
    return ((size_t)rows * 8 + 255) / 256 * 256;
}
inline size_t lmhead_offsets_offset(int64_t rows) {
    return lmhead_draft_offset(rows) + ((size_t)rows * 4 + 255) / 256 * 256;
}
inline size_t lmhead_workspace_bytes(int64_t rows, int32_t num_requests) {
    return lmhead_offsets_offset(rows) + ((size_t)num_requests * 8 + 255) / 256 * 256;
}
// LM-head tiles are 256 columns by at most 256 rows; grid positions run over
// whole groups of kLmheadGroup weight tiles (the kernel's tile order).
constexpr int kLmheadGroup = 4;
// With few row tiles, groups of two: the workgroups that share a weight tile
// then start closer together (544 rows, d = 5,120, 702 -> 692 us; 1,020 rows 1,161 ->
// 1,148; 1,275 rows of 32,000 columns, d = 4,096, 263 -> 262), while 17 row tiles
// want four (4,352 rows 4,772 us, in twos 4,881).
constexpr int kLmheadGroupFew = 2, kLmheadFewRowTiles = 5;
constexpr int64_t lmhead_row_tiles(int64_t rows) { return (rows + 255) / 256; }
// A row tile's height in steps of 32 rows: the rows spread evenly over the row
// tiles (above 128 rows, 5 to 8 steps).
constexpr int64_t lmhead_tile_height(int64_t rows) {
    return ((rows + lmhead_row_tiles(rows) - 1) / lmhead_row_tiles(rows) + 31) / 32;
}
// The least height of any call of at least this many row tiles (that of its
// fewest rows, which grows with the tiles): lower ones need no kernel of theirs.
constexpr int64_t lmhead_least_height(int64_t row_tiles) {
    return lmhead_tile_height(256 * (row_tiles - 1) + 1);
}
hipError_t launch_lmhead_verify(const void* hidden, const void* weight, int64_t d,
                                int64_t vocab, int64_t rows, const CallArgs& a, void* workspace,
                                int num_cus, hipStream_t stream);

// Matrix-core probe: `workgroups` workgroups of the LM-head kernel's shape, each
// running `steps` K steps of its MFMA work on operands held in registers.
hipError_t launch_mfma_probe(const void* operands, int64_t vectors, int64_t workgroups,
                             int64_t steps, uint32_t* out, hipStream_t stream);

// Read probe: `rows` workgroups each streaming `row_bytes` (a multiple of 16)
// from a 16-byte aligned buffer.
hipError_t launch_read_probe(const void* buf, int64_t rows, int64_t row_bytes, uint32_t* out,
                             hipStream_t stream);

}  // namespace asd
