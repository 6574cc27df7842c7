// Host build of the choice of K1's kernels, for tests/test_scale_rules.py.
#include "../paper_2609_05419_amd/csrc/scale_rules.h"

extern "C" {
int t_direct_hold(long k, int two_sources) { return o2m::direct_hold(k, two_sources != 0); }
int t_direct_rule(long entry_bytes, int cs, long k, int two_sources, long rows, long cols) {
    return o2m::direct_rule((size_t)entry_bytes, cs != 0, k, two_sources != 0, rows, cols);
}
}
