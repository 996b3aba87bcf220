// mtgp_split.hpp -- segment lengths of split requests (no HIP).
//
// A stream's jump powers are cached by segment length, so both rules below
// give lengths on coarse grids: a request's length then names one of few
// segment lengths, whose powers are built once.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace mtgp {

// Segment length for a target of v outputs: v rounded down to m * 2^e with
// m in {4, 5, 6, 7} (at most 20% short), at least 256.  The coarse grid
// keeps a stream's segment length, and so its cached jump polynomials, the
// same from batch to batch when the target moves a little; whole 256-word
// multiples keep every segment's stores line-aligned.
inline uint64_t segment_length(uint64_t v) {
    if (v < 1024) return std::max<uint64_t>(256, v / 256 * 256);
    const int e = 63 - __builtin_clzll(v) - 2;  // v / 2^e in [4, 8), e >= 8
    return (v >> e) << e;
}

// Groups: several segments of one narrow stream run together on one wave,
// where a whole wave's window of a short state would be cut into tiny chunks
// per residue class.  W <= 32: 2^group_log(W) segments, each on
// 64 >> group_log(W) lanes; W > 32: every lane takes its class of each of
// GROUP_ROWS segments.
constexpr int group_log(uint32_t W) { return W <= 8 ? 3 : W <= 16 ? 2 : W <= 32 ? 1 : 0; }
constexpr int GROUP_ROWS = 4;
constexpr int group_members(uint32_t W) { return W <= 32 ? 1 << group_log(W) : GROUP_ROWS; }

// Least outputs of a member: it pays a jump, about the time of 4,000 outputs
// at N = 101, and it takes at least the tuning's floor of dependent steps (a
// step being the time of a wide step, 0.4 us, in which a member makes 8 to 18
// outputs for W <= 16 and about W / 2 above).
constexpr uint64_t GROUP_MIN_LSEG = 8192;
inline uint64_t group_least(uint32_t W, int floor_steps) {
    return std::max<uint64_t>(GROUP_MIN_LSEG, (uint64_t)std::max(8u, W / 2) *
                                                  (uint64_t)std::max(0, floor_steps));
}

// Whether a request has members enough for groups: at least half of a group
// busy, nearly all of it where W > 32 (all rows are computed, and the wave
// alone is not much slower).
inline bool group_long_enough(uint32_t W, uint64_t count, int floor_steps) {
    const int n = group_members(W);
    const uint64_t least = group_least(W, floor_steps);
    return W > 32 ? count > (uint64_t)(n - 1) * least
                  : count >= (uint64_t)std::max(2, n / 2) * least;
}

// Segment length of a request cut into groups, for at most `item` outputs a
// group as far as group_least allows.  One or two groups share the request
// evenly, rounded up to m * 2^e, m in {4, 5, 6, 7} (at most a quarter long);
// more take whole groups of `item`, whatever the request's length, and the
// last may be short.
inline uint64_t group_length(uint32_t W, uint64_t count, uint64_t item, int floor_steps) {
    const uint64_t n = (uint64_t)group_members(W), least = group_least(W, floor_steps);
    const uint64_t items = (count + item - 1) / item;
    const uint64_t v =
        std::max(least, items > 2 ? item / n : (count + items * n - 1) / (items * n));
    const int e = 63 - __builtin_clzll(v) - 2;  // v / 2^e in [4, 8)
    return ((v + (1ull << e) - 1) >> e) << e;
}

}  // namespace mtgp
