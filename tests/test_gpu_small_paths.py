"""GPU parity of the kernels' paths for small and ragged problems with the CPU
oracle, whole outputs bit for bit (every output is one correctly rounded
value, so there is no tolerance)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from conftest import same_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def o2m():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_05419_amd as lib
    return lib


def to_dev(x):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(x).T)).to(DEV).t()


def padded(x, pad):
    """to_dev with a leading dimension of rows + pad."""
    rows, cols = x.shape
    buf = torch.full((cols, rows + pad), float("nan"), dtype=torch.from_numpy(x).dtype, device=DEV)
    buf[:, :rows] = to_dev(x).t()
    return buf[:, :rows].t()


def host(t):
    torch.cuda.synchronize()
    return np.asfortranarray(t.cpu().numpy())


def op_of(x, t):
    return x if t == "N" else x.T if t == "T" else x.conj().T


# ------------------------------------------------------------------ residues
# Fragments are 16 rows x 64 k: sizes one below, at and one above both; one
# fragment row with padding beside it; the moduli split in parts (fewer than
# 2048 waves, 768 with one digit) at odd counts, with a hybrid set cut inside
# its 2M and 3M moduli; the two operands' digit counts apart (N = 13, k = 65 and N = 26, k = 17: two
# launches); fp32 pairs with an odd row or k at the edge, and no pairs (odd
# leading dimension); clamped indices must not read the NaN beyond the operand.
RESIDUES = [
    # call, m, n, k, N, rule, transa, transb, pad
    ("z", 15, 17, 63, 16, "max", "N", "N", 1),
    ("z", 16, 16, 64, 16, "cs", "T", "N", 0),
    ("z", 17, 15, 65, 7, "max", "C", "T", 3),
    ("z", 1, 1, 1, 3, "max", "N", "N", 0),
    ("z", 33, 1, 129, 26, "cs", "N", "T", 2),
    ("z", 40, 50, 65, 13, "max", "N", "N", 0),
    ("z", 40, 50, 17, 26, "max", "N", "N", 0),
    ("z", 30, 70, 70, 31, "max", "T", "C", 0),
    ("c", 17, 31, 65, 8, "max", "N", "N", 1),
    ("c", 33, 15, 63, 8, "cs", "T", "T", 1),
    ("c", 31, 47, 127, 5, "max", "N", "C", 2),
    ("c", 16, 48, 66, 8, "max", "C", "N", 2),
    ("z", 120, 9, 3900, 5, "max", "N", "N", 0),     # one digit, rows up to 64-row tiles: 732 waves,
    ("z", 140, 9, 3900, 5, "max", "N", "T", 1),     # and 976
]


@pytest.mark.parametrize("case", RESIDUES, ids=["-".join(str(v) for v in c) for c in RESIDUES])
def test_residue_edges(o2m, case):
    call, m, n, k, N, rule, ta, tb, pad = case
    dt = np.complex64 if call == "c" else np.complex128
    a = W.complex_matrix(*((m, k) if ta == "N" else (k, m)), seed=900 + m, dist="phi", phi=1.0, dtype=dt)
    b = W.complex_matrix(*((k, n) if tb == "N" else (n, k)), seed=901 + n, dist="phi", phi=1.0, dtype=dt)
    fn, ref = (o2m.cgemm_2m_op, O.oq_cgemm) if call == "c" else (o2m.zgemm_2m_op, O.oq_zgemm)
    got = host(fn(padded(a, pad), padded(b, pad), ta, tb, n_moduli=N, scaling=rule))
    assert same_bits(got, ref(op_of(a, ta), op_of(b, tb), N, scaling=rule))


@pytest.mark.parametrize("n,k,N,rule", [(17, 64, 16, "max"), (16, 63, 11, "cs"), (31, 129, 18, "max"), (1, 1, 16, "cs"),
                                        (33, 131, 5, "max"), (15, 255, 9, "cs")])
def test_residue_edges_symmetric(o2m, n, k, N, rule):
    """Rank-2k sources in one launch, and the real split with odd k (its
    imaginary half ends one column before its k does)."""
    a, b = (W.complex_matrix(n, k, s, dist="phi", phi=1.0) for s in (71, 72))
    ra, rb = (W.real_matrix(n, k, s, dist="phi", phi=1.0) for s in (73, 74))
    tri = np.tril_indices(n)
    for got, ref in ((o2m.zher2k_2m(padded(a, 1), padded(b, 2), n_moduli=N, scaling=rule), O.oq_zher2k(a, b, N, scaling=rule)),
                     (o2m.dsyr2k_2m(padded(ra, 1), padded(rb, 2), n_moduli=N, scaling=rule), O.oq_dsyr2k(ra, rb, N, scaling=rule)),
                     (o2m.dsyrk_2m(padded(ra, 1), n_moduli=N, scaling=rule), O.oq_dsyrk(ra, N, scaling=rule))):
        assert same_bits(host(got)[tri], np.asarray(ref)[tri])


# ------------------------------------------------------------- fresh symmetric outputs
@pytest.mark.parametrize("uplo", ["L", "U"])
@pytest.mark.parametrize("n,k", [(1, 3), (31, 5), (32, 8), (33, 7), (530, 4)])
def test_fresh_symmetric_output_is_zero_elsewhere(o2m, n, k, uplo):
    """The whole fresh output: the triangle as the oracle has it, +0 in the
    other one, though the memory held NaN; through the binding, and into a
    buffer of NaN with ldc = n + 3, whose rows beyond n stay as they were.
    Sizes around a 32 x 32 tile and beyond one super-tile (512)."""
    a, b = (W.complex_matrix(n, k, s, dist="phi", phi=0.5) for s in (81, 82))
    ra, rb = (W.real_matrix(n, k, s, dist="phi", phi=0.5) for s in (83, 84))
    dev = {"h": (to_dev(a),), "s": (to_dev(ra),), "x": (to_dev(a), to_dev(b)), "y": (to_dev(ra), to_dev(rb))}
    for op, call, ref, dt in (("h", o2m.zherk_2m, O.oq_zherk(a, 16), np.complex128),
                              ("s", o2m.dsyrk_2m, O.oq_dsyrk(ra, 16), np.float64),
                              ("x", o2m.zher2k_2m, O.oq_zher2k(a, b, 16), np.complex128),
                              ("y", o2m.dsyr2k_2m, O.oq_dsyr2k(ra, rb, 16), np.float64)):
        buf = torch.full((n, n + 3), float("nan"), dtype=dev[op][0].dtype, device=DEV)
        A, B = dev[op][0], dev[op][-1]
        st = o2m._L.o2m_sym_fresh(op.encode(), uplo.encode(), n, k, A.data_ptr(), n, B.data_ptr(), n, buf.data_ptr(),
                                  n + 3, 16, 0, torch.cuda.current_stream().cuda_stream)
        assert st == 0
        torch.cuda.synchronize()
        assert torch.isnan(buf[:, n:].real).all()
        low = np.tril(np.asarray(ref))             # the oracle's lower triangle
        want = low if uplo == "L" else np.triu(low.conj().T)
        keep = np.tril(np.ones((n, n), bool)) if uplo == "L" else np.triu(np.ones((n, n), bool))
        for got in (host(buf[:, :n].t()), host(call(*dev[op], uplo=uplo))):
            assert np.array_equal(got[keep], want[keep])
            assert same_bits(got[~keep], np.zeros(int((~keep).sum()), dt))


# ------------------------------------------------------------------ exponents
def _special(x, rule):
    """Rows that decide an exponent: zero, one subnormal, one huge beside one
    tiny, and (Cauchy-Schwarz) a sum of squares at a power of 4."""
    from cs_inputs import straddle_vector
    m, k = x.shape
    x[0, :] = 0
    if m > 3:
        x[1, :] = 0
        x[1, k // 2] = 5e-310j if x.dtype == np.complex128 else 1e-42j
        x[2, 0] = 1e30
        x[2, k - 1] = 1e-30
    if rule == "cs" and m > 5 and k >= 192:
        x[4, :] = straddle_vector(k, "low", dtype=x.dtype)
        x[5, :] = straddle_vector(k, "high", dtype=x.dtype)
    return x


# The direct kernel takes 4 rows per workgroup, 8 from 960 rows and 16 from 1920
# (not complex fp64 with k <= 1024), 64 entries of a row per round, 1, 4, 8 or
# 16 rounds held in registers (k <= 64, 256, 512, 1024), and calls up to 16384
# entries per row, 16384 + 16 n rows (Cauchy-Schwarz) and 24576 + 4 n (max);
# past that the chunked scans run (Cauchy-Schwarz rule: also between columns
# alone past 3584 entries, and where a row scan has 8 columns per thread).
@pytest.mark.parametrize("rule", ["max", "cs"])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (15, 17, 63), (16, 16, 64), (17, 15, 65), (33, 31, 1024), (18, 20, 1025),
                                   (700, 263, 20), (959, 964, 9), (1915, 18, 1026), (6, 7, 16384), (7, 6, 16385), (2, 2, 0),
                                   (17, 6, 256), (6, 17, 257), (18, 5, 512), (5, 18, 513),
                                   (16416, 2, 3), (16417, 2, 3), (24584, 2, 3), (24585, 2, 3)])
def test_exponents(o2m, m, n, k, rule):
    a = _special(W.complex_matrix(m, k, 41, dist="phi", phi=2.0), rule) if k else np.zeros((m, 0), np.complex128)
    b = _special(W.complex_matrix(n, k, 42, dist="phi", phi=2.0), rule).T if k else np.zeros((0, n), np.complex128)
    b = np.asfortranarray(b)
    _, E, F = o2m.zgemm_2m_residues(to_dev(a), to_dev(b), n_moduli=16, scaling=rule)
    if k:
        E0, _, F0, _ = O.exponents(a, b, rule)
        assert np.array_equal(E.cpu().numpy(), E0) and np.array_equal(F.cpu().numpy(), F0)
    else:
        assert not E.any() and not F.any()
        return
    for ta, tb in (("N", "N"), ("T", "T")):
        A, B = a if ta == "N" else np.asfortranarray(a.T), b if tb == "N" else np.asfortranarray(b.T)
        got = host(o2m.zgemm_2m_op(padded(A, 1), padded(B, 1), ta, tb, n_moduli=16, scaling=rule))
        assert same_bits(got, O.oq_zgemm(a, b, 16, scaling=rule))
    af, bf = (_special(W.complex_matrix(r, k, 43, dist="phi", phi=1.0).astype(np.complex64), rule) for r in (m, n))
    bf = np.asfortranarray(bf.T)
    assert same_bits(host(o2m.cgemm_2m(to_dev(af), to_dev(bf), n_moduli=8, scaling=rule)), O.oq_cgemm(af, bf, 8, scaling=rule))


@pytest.mark.parametrize("rule", ["max", "cs"])
@pytest.mark.parametrize("n,k", [(17, 65), (965, 9), (33, 1030), (18, 8192), (18, 8193), (20, 16385)])
def test_exponents_symmetric(o2m, n, k, rule):
    """Both sources of a rank-2k update count towards the limit (8192 each)."""
    a, b = (_special(W.complex_matrix(n, k, s, dist="phi", phi=1.0), rule) for s in (51, 52))
    b[4:6, :] = 0                                        # the straddling rows of [A | B] are A's
    ra, rb = a.real.copy(order="F"), b.real.copy(order="F")
    tri = np.tril_indices(n)
    for got, ref in ((o2m.zherk_2m(to_dev(a), scaling=rule), O.oq_zherk(a, 16, scaling=rule)),
                     (o2m.zher2k_2m(to_dev(a), to_dev(b), scaling=rule), O.oq_zher2k(a, b, 16, scaling=rule)),
                     (o2m.dsyrk_2m(to_dev(ra), scaling=rule), O.oq_dsyrk(ra, 16, scaling=rule)),
                     (o2m.dsyr2k_2m(to_dev(ra), to_dev(rb), scaling=rule), O.oq_dsyr2k(ra, rb, 16, scaling=rule))):
        assert same_bits(host(got)[tri], np.asarray(ref)[tri])


@pytest.mark.parametrize("n", [4096, 4097])
def test_exponents_many_rows_of_two_sources(o2m, n):
    """Up to 4096 rows the direct kernel, more the row scans (Cauchy-Schwarz)."""
    k = 5
    a, b = (_special(W.complex_matrix(n, k, s, dist="phi", phi=1.0), "max") for s in (53, 54))
    got = host(o2m.zher2k_2m(to_dev(a), to_dev(b), scaling="cs"))
    rng = np.random.default_rng(n)
    ent = [(0, 0), (n - 1, 0), (n - 1, n - 1), (2, 1)]
    ent += [(max(i, j), min(i, j)) for i, j in rng.integers(0, n, (300, 2)).tolist()]
    assert same_bits(np.array([got[i, j] for i, j in ent]), O.oq_zher2k(a, b, 16, entries=ent, scaling="cs"))


@pytest.mark.parametrize("k", [40, 1030, 16390])
@pytest.mark.parametrize("rule", ["max", "cs"])
def test_exponents_nonfinite(o2m, k, rule):
    """Inf or NaN in a row or column: NaN there, the status bit, the rest exact."""
    m, n = 19, 21
    a, b = W.complex_matrix(m, k, 61), W.complex_matrix(k, n, 62)
    clean = O.oq_zgemm(a, b, 16, scaling=rule)
    a[3, k - 1] = complex(np.nan, 1.0)
    a[17, 0] = complex(0.0, -np.inf)
    b[k // 2, 20] = complex(np.inf, 0.0)
    o2m.get_status()
    got = host(o2m.zgemm_2m(to_dev(a), to_dev(b), n_moduli=16, scaling=rule))
    assert o2m.get_status() == o2m.STATUS_NONFINITE
    bad = np.zeros((m, n), bool)
    bad[[3, 17], :] = True
    bad[:, 20] = True
    assert np.isnan(got[bad].real).all() and np.isnan(got[bad].imag).all()
    assert same_bits(got[~bad], clean[~bad])


@pytest.mark.parametrize("m,n,k", [(17, 15, 65), (3, 5, 16384), (5, 3, 16385)])
def test_gauss_maxima(o2m, m, n, k):
    """The bound check reads the maxima of whichever kernel found them."""
    A, B = W.gauss_matrix(m, k, 7, lo=-50, hi=50), W.gauss_matrix(k, n, 8, lo=-50, hi=50)
    dA, dB = (torch.from_numpy(x).to(DEV).transpose(0, 1) for x in (A, B))
    o2m.get_status()
    got = o2m.gauss_gemm_2m(dA, dB, n_moduli=4).transpose(0, 1).cpu().numpy()
    assert o2m.get_status() == 0 and np.array_equal(got, O.gauss_4m(A, B))
    o2m.gauss_gemm_2m(dA, dB, n_moduli=2)                # M = 56153: the bound is far exceeded
    assert o2m.get_status() == o2m.STATUS_OVERFLOW


# ------------------------------------------------------------------ GEMM tiles
def _gemm_sizes():
    from gemm_shapes import CHAINED, SHAPES
    return [(s, *c) for s, cs in SHAPES.items() for c in cs] + [("chain", *c) for c in CHAINED]


@pytest.mark.parametrize("shape,m,n,k,products", _gemm_sizes())
def test_gemm_tile_shapes(o2m, shape, m, n, k, products):
    """Every tile shape of the int8 GEMM (test_gemm_plan checks that these
    sizes take it): two entries of every 64 x 64 block and the corners."""
    N = 32 if products == 74 else products // 2
    a, b = W.complex_matrix(m, k, 31, dist="phi", phi=0.5), W.complex_matrix(k, n, 32, dist="phi", phi=0.5)
    got = host(o2m.zgemm_2m(to_dev(a), to_dev(b), n_moduli=N))
    rng = np.random.default_rng(m + n)
    ent = [(i, j) for i in (0, m - 1) for j in (0, n - 1)]
    for i in range(0, m, 64):
        for j in range(0, n, 64):
            ent += [(int(rng.integers(i, min(m, i + 64))), int(rng.integers(j, min(n, j + 64)))) for _ in range(2)]
    assert same_bits(np.array([got[i, j] for i, j in ent]), O.oq_zgemm(a, b, N, entries=ent))


@pytest.mark.parametrize("n,k", [(65, 100), (130, 70), (190, 600), (700, 900), (1000, 65)])
def test_gemm_tiles_symmetric(o2m, n, k):
    """The symmetric calls read both operands from one set of planes, written
    up to whole tiles of either side."""
    a = W.complex_matrix(n, k, 33, dist="phi", phi=0.5)
    got = host(o2m.zherk_2m(to_dev(a)))
    rng = np.random.default_rng(n)
    ent = [(i, j) for i in (0, n - 1) for j in (0, n - 1) if i >= j]
    ent += [(max(i, j), min(i, j)) for i, j in rng.integers(0, n, (400, 2)).tolist()]
    assert same_bits(np.array([got[i, j] for i, j in ent]), O.oq_zherk(a, 16, entries=ent))


# ------------------------------------------------------------------ CRT
# One row per thread up to 160 rows or 2^20 entries, four beyond: both sides of
# either line, wave and workgroup edges, two to six limbs.
@pytest.mark.parametrize("m,n,N", [(1, 300, 16), (63, 70, 8), (65, 64, 20), (160, 40, 26), (161, 41, 31), (255, 9, 16),
                                   (257, 9, 18), (1025, 5, 8), (1024, 1024, 8), (1025, 1024, 16), (1030, 1027, 20),
                                   (161, 6600, 26), (1281, 1000, 31), (160, 6600, 16)])
def test_crt_rows(o2m, m, n, N):
    k = 3
    a, b = W.complex_matrix(m, k, 21, dist="phi", phi=1.0), W.complex_matrix(k, n, 22, dist="phi", phi=1.0)
    cols = sorted({0, n // 3, n - 2 if n > 1 else 0, n - 1})
    ent = [(i, j) for j in cols for i in range(m)]
    for dt, fn, ref in ((np.complex128, o2m.zgemm_2m, O.oq_zgemm), (np.complex64, o2m.cgemm_2m, O.oq_cgemm)):
        x, y = a.astype(dt), b.astype(dt)
        out = torch.full((n, m + 3), complex("nan"), dtype=torch.from_numpy(x).dtype, device=DEV)
        got = fn(to_dev(x), to_dev(y), n_moduli=N, out=out[:, :m].t())
        assert torch.isnan(out[:, m:].real).all()                # nothing beyond the rows is written
        assert not torch.isnan(out[:, :m].real).any()            # and every row is
        got = host(got)
        assert same_bits(np.array([got[i, j] for i, j in ent]), ref(x, y, N, entries=ent))


@pytest.mark.parametrize("m,n", [(3, 5), (161, 7), (257, 3), (1030, 1030)])
def test_crt_rows_gauss(o2m, m, n):
    A, B = W.gauss_matrix(m, 4, 23), W.gauss_matrix(4, n, 24)
    dA, dB = (torch.from_numpy(x).to(DEV).transpose(0, 1) for x in (A, B))
    o2m.get_status()
    got = o2m.gauss_gemm_2m(dA, dB, n_moduli=4).transpose(0, 1).cpu().numpy()
    assert o2m.get_status() == 0 and np.array_equal(got, O.gauss_4m(A, B))


# ------------------------------------------------------------------ chunked scans
# Past the direct kernel's rows (16384), with 4 columns per thread in the row
# scans: two operands in one launch (row scan beside column scan, two row scans,
# two column scans), and apart (column pairs of one fp32 operand only).
@pytest.mark.parametrize("call,m,n,k,ta,tb,pad", [("z", 7, 9, 16390, "N", "N", (0, 0)), ("z", 9, 7, 16385, "N", "T", (1, 1)),
                                                  ("z", 6, 65, 16401, "T", "N", (0, 2)), ("z", 65, 6, 16400, "C", "T", (1, 0)),
                                                  ("c", 8, 6, 16386, "N", "N", (0, 0)), ("c", 7, 9, 16387, "T", "N", (1, 1)),
                                                  ("c", 6, 8, 16388, "T", "N", (0, 1)), ("c", 5, 9, 16385, "N", "T", (1, 1))])
def test_scans_of_two_operands(o2m, call, m, n, k, ta, tb, pad):
    dt = np.complex64 if call == "c" else np.complex128
    a = _special(W.complex_matrix(m, k, 11, dist="phi", phi=1.0).astype(dt), "cs")
    b = np.asfortranarray(_special(W.complex_matrix(n, k, 12, dist="phi", phi=1.0).astype(dt), "cs").T)
    A, B = np.asfortranarray(op_of(a, ta)), np.asfortranarray(op_of(b, tb))   # op is its own inverse
    fn, ref = (o2m.cgemm_2m_op, O.oq_cgemm) if call == "c" else (o2m.zgemm_2m_op, O.oq_zgemm)
    got = host(fn(padded(A, pad[0]), padded(B, pad[1]), ta, tb, n_moduli=16, scaling="cs"))
    assert same_bits(got, ref(a, b, 16, scaling="cs"))


def _scan_sizes():
    from scale_shapes import SCANS
    return [c[:6] for c in SCANS]


@pytest.mark.parametrize("call,m,n,k,ta,tb", _scan_sizes())
def test_scans_by_columns_per_thread(o2m, call, m, n, k, ta, tb):
    """Every number of columns per thread of the row scan, beside a column scan
    and a row scan, with plain and non-temporal loads, and long columns
    (test_scale_rules checks that these sizes take them).  All exponents, where
    the hook gives them, and sampled entries, among them the rows and columns
    that the records leave open."""
    from cs_inputs import straddle_vector
    dt = np.complex64 if call == "c" else np.complex128
    a = W.complex_matrix(m, k, 13, dist="phi", phi=1.0).astype(dt)
    b = W.complex_matrix(k, n, 14, dist="phi", phi=1.0).astype(dt)
    wide = dict(exact=(0, 2048), binade=(2048, 2112), stride=2048)     # chunks of 2048 along a column
    if k > 2112:
        a[7, :], a[m - 1, :] = (straddle_vector(k, s, dtype=dt, **({} if ta == "N" else wide)) for s in ("low", "high"))
        b[:, 3], b[:, n - 1] = (straddle_vector(k, s, dtype=dt, **(wide if tb == "N" else {})) for s in ("high", "low"))
    A, B = (to_dev(np.asfortranarray(op_of(x, t))) for x, t in ((a, ta), (b, tb)))
    if call == "z" and ta == tb == "N":
        _, E, F = o2m.zgemm_2m_residues(A, B, n_moduli=16, scaling="cs")
        E0, _, F0, _ = O.exponents(a, b, "cs")
        assert np.array_equal(E.cpu().numpy(), E0) and np.array_equal(F.cpu().numpy(), F0)
    fn, ref = (o2m.cgemm_2m_op, O.oq_cgemm) if call == "c" else (o2m.zgemm_2m_op, O.oq_zgemm)
    N = 8 if call == "c" else 16
    got = fn(A, B, ta, tb, n_moduli=N, scaling="cs")
    rng = np.random.default_rng(m)
    ent = [(i, j) for i in (0, 7, m - 1) for j in (0, 3, n - 1)]
    ent += [(int(i), int(j)) for i, j in zip(rng.integers(0, m, 60), rng.integers(0, n, 60))]
    idx = torch.tensor(ent, device=DEV)
    assert same_bits(got[idx[:, 0], idx[:, 1]].cpu().numpy(), ref(a, b, N, entries=ent, scaling="cs"))
