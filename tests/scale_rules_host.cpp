// Host build of the choice of K1's kernels, for tests/test_scale_rules.py.
#include "../paper_2609_05419_amd/csrc/scale_rules.h"

extern "C" {
int t_direct_hold(long k, int two_sources) { return o2m::direct_hold(k, two_sources != 0); }
int t_direct_rule(long entry_bytes, int cs, long k, int two_sources, long rows, long larger,
                  long cols) {
    return o2m::direct_rule((size_t)entry_bytes, cs != 0, k, two_sources != 0, rows, larger, cols);
}
int t_row_cpt(int rows, int cols) { return o2m::cs_row_cpt(rows, cols); }
// v: mode, columns per thread, pairs, non-temporal, bytes, workgroups of either scan
int t_scans_together(const long *a, const long *b) {
    auto shape = [](const long *v) {
        return o2m::ScanShape{(int)v[0], (int)v[1], v[2] != 0, v[3] != 0, (size_t)v[4], v[5]};
    };
    return o2m::scans_together(shape(a), shape(b));
}
}
