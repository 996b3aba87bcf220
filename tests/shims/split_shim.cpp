// C entry points for tests/test_split_rules.py.
#include "mtgp_split.hpp"

extern "C" {
unsigned long long split_segment_length(unsigned long long v) { return mtgp::segment_length(v); }
int split_group_members(unsigned W) { return mtgp::group_members(W); }
unsigned long long split_group_least(unsigned W, int floor_steps) {
    return mtgp::group_least(W, floor_steps);
}
int split_group_long_enough(unsigned W, unsigned long long count, int floor_steps) {
    return mtgp::group_long_enough(W, count, floor_steps) ? 1 : 0;
}
unsigned long long split_group_length(unsigned W, unsigned long long count,
                                      unsigned long long item, int floor_steps) {
    return mtgp::group_length(W, count, item, floor_steps);
}
}
