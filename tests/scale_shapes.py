"""Sizes that the direct exponent kernel leaves to the scans, shared by the GPU tests of the
chunked scans and the host test of the rules that send them there."""

# call, m, n, k, transa, transb, columns per thread of A's row scan (0: A is
# scanned in columns), whether A's loads are non-temporal (128 MiB and more)
SCANS = [
    ("z", 2100, 45, 2300, "N", "N", 8, False),
    ("z", 3001, 45, 3003, "N", "N", 16, True),        # B's small scan non-temporal beside A's
    ("z", 4099, 45, 4099, "N", "N", 32, True),
    ("z", 45, 2100, 2300, "T", "T", 0, False),        # 45 columns beside 2100 rows
    ("z", 3001, 3001, 900, "N", "T", 4, False),       # two row scans
    ("c", 4099, 45, 4100, "N", "N", 32, True),        # pairs of fp32 columns
    ("c", 3001, 1001, 3002, "N", "N", 16, False),
    ("c", 2901, 1300, 2301, "T", "N", 0, False),      # two column scans, odd leading dimensions
    ("z", 1101, 45, 4101, "N", "N", 8, False),        # within the caches, 8 columns per thread
    ("z", 1101, 33, 4101, "N", "T", 8, False),        # the same, a small row scan apart
    ("c", 45, 30, 3585, "T", "N", 0, False),          # long columns alone
]
# k of rows that the scans' records leave open
RESUMMED_K = 17000          # GEMM calls, ZHERK, DSYRK
RESUMMED_K_RANK2 = 8700     # two sources
