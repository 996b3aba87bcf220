// mtgp_internal.hpp -- declarations shared by the kernels and the host
// library (never installed; the public interface is include/mtgp.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "mtgp_split.hpp"

namespace mtgp {

// Device parameter block: 1024 words (4 KB) per stream.
enum : uint32_t {
    P_MEXP = 0,
    P_N = 1,
    P_POS = 2,
    P_SH1 = 3,
    P_SH2 = 4,
    P_MASK = 5,
    P_W = 6,
    P_SEED = 7,
    P_LIN = 8,     // 1 if the recursion table is GF(2)-linear (rec[i^j] = rec[i]^rec[j])
    P_RB = 9,      // its basis: rec[1], rec[2], rec[4], rec[8] (words 9..12)
    P_REC = 16,
    P_TMP = 32,
    P_FLT = 48,
    // windowed small-step path (linear recursion table, W < 64)
    P_WIN_WN = 64,       // window length (<= N-1)
    P_WIN_E = 65,        // elements per lane and window
    P_WIN_Q = 66,        // lanes per residue class (64 / W)
    P_WIN_ROUNDS = 67,   // cross-lane scan rounds, ceil(log2 q)
    P_WIN_MAT = 128,     // nibble tables of M^(E*2^r): [round][nibble][16]
    P_GRP_MAT = 768,     // groups with several lanes per class: M^(8*2^r), r < 2
    P_WORDS = 1024,      // 4 KB per stream
};
constexpr int WIN_EMAX = 8;
constexpr int WIN_MAXROUNDS = 5;
constexpr int WIN_MAT_WORDS = 128;   // 8 nibbles x 16 entries

// Groups (mtgp_split.hpp) only for N <= 128 (several states fit a wave's LDS)
// and linear recursion tables.
constexpr bool has_groups(int N) { return N <= 128; }
constexpr int GROUP_E = 8;           // most elements per lane and window
constexpr int GROUP_ROUNDS = 2;      // scan rounds (W = 2: four lanes per class)

// BatchItem.mode bits
enum : uint32_t {
    MODE_F32 = 1u,     // float32 output (else uint32)
    MODE_RAW = 2u,     // also store the raw words x_0 .. x_{N+count-1} at raw
    MODE_VERIFY = 4u,  // compare the end state with verify[0..N); a mismatch
                       // marks the item's request record as failed
    MODE_FIXUP = 8u,   // request check (last launch of a batch): regenerate
                       // the request from its record if a segment failed,
                       // then raise `flag`
    MODE_GROUP = 16u,  // segments of a split request, or a whole one (GroupItem)
};

// Request record (64 bytes) of a request split by jump-ahead: its segments
// mark `failed` when a check fails, and the batch's last launch (after
// every segment has finished, so no later store can land on its outputs)
// regenerates such a request in order from `orig`.
struct ReqRec {
    uint32_t failed;     // nonzero once a segment's end state missed the next start
    uint32_t stream;
    uint32_t mode;       // MODE_F32 or 0
    uint32_t reserved0;
    uint64_t count;      // outputs of the whole request
    uint64_t out;        // device address of its first output
    uint64_t orig;       // N words: the stream's state when the request starts
    uint64_t row;        // where the request's final state goes
    uint64_t reserved[2];
};
static_assert(sizeof(ReqRec) == 64, "ReqRec layout");

// Device work-list entry (80 bytes): advance a stream from state_in by
// `count` outputs written to `out`, store the end state at state_out.
struct BatchItem {
    uint32_t stream;
    uint32_t mode;
    uint64_t count;
    uint64_t out;        // device address of the outputs
    uint64_t state_in;   // N words
    uint64_t state_out;  // N words, or 0
    uint64_t raw;        // MODE_RAW destination
    uint64_t verify;     // MODE_VERIFY reference state
    uint64_t rec;        // the request's ReqRec (MODE_VERIFY, MODE_FIXUP), or 0
    uint64_t flag;       // 0, or a host-mapped uint32 set to 1 when the request is done
    uint64_t reserved;
};
static_assert(sizeof(BatchItem) == 80, "BatchItem layout");

// A BatchItem with MODE_GROUP: segments first .. first + n - 1 of a split
// request (a whole request: lseg = count, prefix = 0).  Segment k covers
// outputs [start, end) of the request with start = prefix (k = 0) or k * lseg
// and end = min(count, (k+1) * lseg); its start state is states + k * N words,
// and its end state must equal segment k+1's start state, or goes to state_out
// when it ends the request.
struct GroupItem {
    uint32_t stream;
    uint32_t mode;
    uint64_t count;      // of the whole request
    uint64_t out;        // of the whole request
    uint64_t states;
    uint64_t state_out;
    uint64_t lseg;
    uint32_t first, n;
    uint64_t rec;
    uint64_t flag;       // 0: the request's check item raises it
    uint64_t prefix;     // outputs the prefix item makes
};
static_assert(sizeof(GroupItem) == sizeof(BatchItem) &&
                  offsetof(GroupItem, flag) == offsetof(BatchItem, flag) &&
                  offsetof(GroupItem, mode) == offsetof(BatchItem, mode),
              "GroupItem layout");

// Batch workspace header (256 bytes, never part of an uploaded plan):
//   word 0, 1   claim counters of the prefix and segment launches
//   word 2      requests regenerated after a failed segment check
//   word 3      entries written to the log (may exceed HDR_LOG_MAX)
//   word 4..11  stream ids of the first HDR_LOG_MAX such requests
//   word 12     unused
//   word 13, 14 tag: a 64-bit value derived from the workspace address; a
//               header without it (fresh or reused memory) is cleared by
//               the first launch of the next call
//   word 15     claim counter of the jump blocks
//   byte 64..95 phase timestamps (64-bit: start, after the prefix and
//               jump launch, after the segments, end)
//   word 24     claim counter of the whole-request list when it runs beside
//               the prefix and jump launch
//   word 25     claim counter of the items that whole workgroups run
constexpr int HDR_ERR = 2;
constexpr int HDR_LOG_MAX = 8;
constexpr int HDR_ERR_WORDS = 2 + HDR_LOG_MAX;  // words HDR_ERR .. HDR_ERR + 9
constexpr int HDR_TAG = 13;
constexpr int HDR_J_CLAIM = 15;
constexpr int HDR_W_CLAIM = 24;
constexpr int HDR_B_CLAIM = 25;
constexpr size_t HDR_STAMP_BYTE = 64;
constexpr size_t HDR_BYTES = 256;

// Jump block (48 bytes): up to JUMP_BLOCK jumps of one stream, each
// out_j[m] = XOR_{i < nbits, g_j,i = 1} raw[1 + i + m] for m < this block's m.
// A state longer than jump_words(N) is covered by several blocks (pass p
// takes the words from p * jump_words(N) on, its raw and out pointers moved
// by as many), so that the passes of a jump run on different workgroups.
constexpr int JUMP_BLOCK = 8;
struct JumpBlock {
    uint64_t raw;          // words x_0, x_1, ... of a stream (nbits + m + 1 of them)
    uint64_t poly;         // jump j's coefficients, 32 per word, at poly + j * poly_stride;
                           // zero from nbits up to the end of the last word
    uint64_t out;          // jump j's m words at out + j * out_stride
    uint32_t poly_stride;  // words, ceil(nbits / 32)
    uint32_t out_stride;   // words
    uint32_t nbits;
    uint32_t m;
    uint32_t n_jumps;      // 1 .. JUMP_BLOCK
    uint32_t dep;          // index of the prefix item that writes raw
};
static_assert(sizeof(JumpBlock) == 48, "JumpBlock layout");
// Tiles of 128 output words a block evaluates at once, and the words of a
// pass: the state cut evenly into as few passes as four tiles allow (three
// at N = 351 and 726, where they fit better).
constexpr int JUMP_TILE = 128;
constexpr int jump_tiles(int N) { return N <= 128 ? 1 : N <= 768 ? 3 : 4; }
constexpr int jump_passes(int N) {
    return (N + JUMP_TILE * jump_tiles(N) - 1) / (JUMP_TILE * jump_tiles(N));
}
constexpr int jump_words(int N) {
    return ((N + jump_passes(N) - 1) / jump_passes(N) + 3) / 4 * 4;
}

struct LaunchArgs {
    const uint32_t *params;
    const BatchItem *items;  // nullptr: plain mode, item i is stream i
    uint32_t n_items;
    uint32_t *plain_states;  // plain mode: state rows, outputs, count, dtype
    uint32_t plain_stride;
    uint32_t *plain_out;
    uint64_t plain_count;
    uint32_t plain_mode;
    uint32_t *counter;
    uint32_t *err;           // header word HDR_ERR (repair count, then the log)
    uint32_t win_below;      // window path for eligible streams with W below this
    int groups_per_cu;       // persistent launches: at most this many groups per CU (0 = occupancy)
    bool persistent;
    bool groups;             // launch_variant: items may carry MODE_GROUP
    int num_cus;
    void *stream;
};

struct VariantInfo {
    int tps, k, wpb;
    size_t lds_bytes[2];     // per workgroup, without and with room for groups
};

int variant_count(int n_words, VariantInfo *out, int max_out);
hipError_t launch_variant(int n_words, int tps, int k, int wpb, const LaunchArgs &a,
                          bool *found);
// Jump blocks alone (their raw words are there), for state length n_words.
hipError_t launch_jump(int n_words, const JumpBlock *blocks, uint32_t n_blocks, int num_cus,
                       hipStream_t s);
// Launches of the prefix kernel (persistent; items may carry MODE_RAW) and,
// below, of the request-check kernel (MODE_FIXUP items) for state length
// n_words (a.win_below applies).
hipError_t launch_prefix(int n_words, const LaunchArgs &a);
// Plain calls of few streams (one wave per stream, a.win_below applies).
hipError_t launch_few(int n_words, const LaunchArgs &a);
// LDS bytes of one prefix-and-jump workgroup.
size_t prefix_jump_lds_bytes(int n_words);
// Prefix items (nP, one wave each) and jump blocks (nJ; block b waits for
// pflag[b.dep]) in one persistent launch.
hipError_t launch_prefix_jumps(int n_words, const BatchItem *prefix, uint32_t nP,
                               const JumpBlock *jumps, uint32_t nJ, uint32_t *pflag,
                               const uint32_t *params, uint32_t *hdr, uint32_t win_below,
                               int num_cus, hipStream_t s);
// Segment launch of a batch that leaves the chip nearly empty: the first
// n_wide items by workgroups of 256, the others by waves (a.counter; the
// wide items' counter is `wide_counter`).  Which items are wide: W at least
// WIDE_MIN_W.
constexpr uint32_t WIDE_MIN_W = 128;
constexpr bool has_wide(int N) { return N > (int)WIDE_MIN_W; }
hipError_t launch_sparse(int n_words, const LaunchArgs &a, uint32_t n_wide,
                         uint32_t *wide_counter);
hipError_t launch_check(int n_words, const LaunchArgs &a);
int variant_slots_per_cu(int n_words, int tps, int k, int wpb, bool groups);
hipError_t launch_seed(const uint32_t *params, uint32_t *states, uint32_t stride,
                       uint32_t n_streams, hipStream_t s);
hipError_t launch_reset(uint32_t *counter, hipStream_t s);
// Zeroes n consecutive words with a small kernel (no memset node, so it is
// safe inside captured graphs).
hipError_t launch_clear(uint32_t *p, uint32_t n, hipStream_t s);
// First launch of every batch call: zeroes the claim counters; zeroes the
// repair count and log when clear_errors is set or the header lacks `tag`
// (then also the timestamps), and writes the tag.
hipError_t launch_header(uint32_t *hdr, uint64_t tag, bool clear_errors, hipStream_t s);
hipError_t launch_stamp(uint64_t *dst, hipStream_t s);
// Device address of the current GPU's static scratch array (looked up once
// per device).
hipError_t scratch_address(void **out);
hipError_t launch_workgroup(const uint32_t *params, uint32_t *states, uint32_t stride,
                            uint32_t n_streams, uint64_t count, uint32_t *out, uint32_t f32,
                            uint32_t threads, uint32_t n_words, hipStream_t s);
hipError_t launch_screen(const uint32_t *out, uint32_t n_streams, uint64_t count, uint32_t lo,
                         uint32_t hi, uint32_t bins, uint64_t *counts, hipStream_t s);
// Piece of a result copy: `bytes` (at most COPY_PIECE) from src to dst.
constexpr uint64_t COPY_PIECE = 64 << 10;
struct CopyPiece {
    uint64_t src, dst, bytes;
};
// Copies n pieces; the list may lie in host-mapped memory.
hipError_t launch_copy(const CopyPiece *pieces, uint32_t n, hipStream_t s);
hipError_t launch_fill(uint32_t *out, uint64_t n_words, uint32_t value, int num_cus,
                       hipStream_t s);

}  // namespace mtgp
