// K1: which calls find their exponents straight from the operands
// (exponents_direct, k_scale.hip), and in which of its forms; which scans of
// two operands go out in one launch.
#pragma once

#include <stddef.h>

namespace o2m {

// Entries of an operand row that a thread holds in registers between the
// maximum and the Cauchy-Schwarz sum: rows of up to 64 times as many.
constexpr int kHold = 16;
constexpr long kDirectK = 16384;                     // entries per operand row, both sources
constexpr size_t kDirectBytes = size_t(72) << 20;    // of both operands
constexpr long kDirectRowsCs = 16384, kDirectRowsPerColumnCs = 16;
constexpr long kDirectRowsMax = 24576, kDirectRowsPerColumnMax = 4;
constexpr long kDirectRowsTwo = 4096;                // Cauchy-Schwarz rule, two sources
constexpr long kDirectColumnK = 3584;                // Cauchy-Schwarz rule, columns only

// Entries held per thread, 64 threads to a row: 1, 4, 8 or 16 (each its own
// form of the kernel, so that a short row costs no more than its own rounds),
// or 0 for a row that is read again: one longer than all of these, or one
// with two sources (rank-2k updates).
inline int direct_hold(long k, bool two_sources) {
    if (two_sources || k > 64 * kHold) return 0;
    return k <= 64 ? 1 : k <= 256 ? 4 : k <= 512 ? 8 : kHold;
}

// Columns per thread of the row-mode scan: 32 (a workgroup covers 64 rows x
// 128 columns), fewer (down to 4) when the grid would otherwise hold fewer
// than ~2048 workgroups (small matrices).
inline int cs_row_cpt(int rows, int cols) {
    const long rb = (rows + 63) / 64;
    int cpt = 32;
    while (cpt > 4 && rb * ((cols + 4 * cpt - 1) / (4 * cpt)) < 2048) cpt >>= 1;
    return cpt;
}

// rows: operand rows that are rows of a column-major matrix (of A, or of a
// transposed B), larger: of those, the ones of the operand that has more; cols:
// those that are its columns.
//
// The direct kernel takes calls whose operands the caches can hold for its
// second reading (2048 x 2048 x 1024, 64 MiB: 21.4 us against the chunked
// scans' 31.2; 1500 x 1500 x 2000, 92 MiB: 39.8 against 39.5; 2048^3, 128 MiB:
// 52.7 against 45.7), up to a row length where a workgroup's walk along its
// rows alone evens out with the scans' parallel chunks (64 x 64 x 16000: 68.4
// against 72.4; 300 x 300 x 4096: 23.2 against 33.6).
//
// It spends a wave's 64 lanes on every operand row however short, where a row
// scan gives one lane of a wave to each of 64 rows: many rows go to the scans.
// Columns count the other way, since the column scans spend 256 threads on
// each.  (Scale phase in us, direct against the scans, m x n x k complex fp64,
// fp32 in brackets.  Cauchy-Schwarz rule: 16384 x 1 x 16 10.6 and 11.0 (12.6,
// 11.1), 16384 x 1 x 300 fp32 19.3, 18.5, 65536 x 1 x 16 25.4 and 17.8 (32.3,
// 16.8); 65536 x 2048 x 16 28.4 and 23.9 (33.6, 22.9), 65536 x 8192 x 16 31.2
// and 38.9 (39.0, 40.2), 131072 x 8192 x 16 54.8 and 91.8 (74.5, 102).  Max
// rule: 24576 x 1 x 16 10.3 and 14.3 (13.9, 15.0), 65536 x 1 x 16 17.3 and 15.9
// (25.2, 15.2), 65536 x 8192 x 16 22.5 and 26.1 (31.3, 25.3).  Rank-2k updates
// under the Cauchy-Schwarz rule, whose two sources are both read again: ZHER2K
// 8192 x 16 12.0 and 11.9, 8192 x 64 21.1 and 15.6.)
//
// Under the Cauchy-Schwarz rule, which reads a row of more than 1024 entries
// twice, the scans are the faster ones in two more places (scale phase again).
// Where a row scan has 8 columns per thread or more, and so half the records to
// combine or fewer: DSYRK 1000 x 4000 23.7 and 28.8 (4 columns), 1500 x 3000
// 29.7 and 21.7, 600 x 8000 45.3 and 30.1, ZHERK 1100 x 4100 34.8 and 28.3,
// DSYR2K 800 x 5500 78.0 and 38.7; least from 1920 rows on, where the direct
// kernel has 16 rows per workgroup (2000 x 3000 22.3 and 22.4, 3000 x 2500 30.9
// and 24.8).  And between columns alone, whose chunks leave few records: 64 x
// 64 x 2560 complex fp64 13.4 and 11.0, 4000 15.4 and 11.2, 16384 47.0 and 17.0;
// fp32 64 x 64 x 4000 14.1 and 11.5, 1000 x 1000 x 4000 30.4 and 26.3, but 800 x
// 800 x 3500 20.0 and 22.6.
inline bool direct_rule(size_t entry_bytes, bool cs, long k, bool two_sources, long rows, long larger, long cols) {
    const size_t per_row = (size_t)k * (two_sources ? 2 : 1);
    const size_t bytes = entry_bytes * per_row * ((size_t)rows + (size_t)cols);
    const long most = !cs ? kDirectRowsMax + kDirectRowsPerColumnMax * cols
                    : two_sources ? kDirectRowsTwo : kDirectRowsCs + kDirectRowsPerColumnCs * cols;
    if (cs && rows == 0 && k > kDirectColumnK) return false;
    if (cs && larger > 0 && k > 64 * kHold && k <= kDirectK && cs_row_cpt((int)larger, (int)k) > 4) return false;
    return per_row <= (size_t)kDirectK && bytes <= kDirectBytes && rows <= most;
}

// One operand of a chunked scan (cs_scan_kernel).
struct ScanShape {
    int mode;              // 0: rows of a column-major matrix, 1: its columns
    int cpt;               // columns per thread in row mode (column mode: 4, the least)
    bool pairs, nt;        // 16-byte pairs, non-temporal loads
    size_t bytes;          // of the operand
    long groups;           // workgroups
};
constexpr size_t kBesideBytes = size_t(16) << 20;   // an operand that may adapt to the other
constexpr long kBesideGroups = 2048;

// Whether the scans of a and b can share a launch, and gain by it.  The kernel
// of a row scan of 32 columns per thread holds two workgroups per CU; a column
// scan beside it is held to as many.  That suits a small one (scale phase
// together and apart: 4096 x 96 x 4096 64.1 and 68.5 us, 150000 x 2000 x 64 75.7
// and 77.5), but not a large operand, nor one of many short columns (150000 x
// 3000 x 64 80.8 and 80.1, 150000 x 8192 x 64 106 and 92.5).
inline bool scans_together(const ScanShape &a, const ScanShape &b) {
    if (a.mode == b.mode) {
        if (a.mode == 0 ? a.cpt != b.cpt : a.pairs != b.pairs) return false;
    } else if (a.cpt >= 32 || b.cpt >= 32) {
        const ScanShape &c = a.mode == 1 ? a : b;
        if (c.bytes >= kBesideBytes || c.groups > kBesideGroups) return false;
    }
    // a small operand may go past the caches along with a large one
    return a.nt == b.nt || (a.bytes < b.bytes ? a.bytes : b.bytes) < kBesideBytes;
}

}  // namespace o2m
