// K2: quantization, residues and the 2M pre step (Algorithm 1 steps 3-4,
// eq. 2m-pre).
//
// For every entry x = a 2^(p - E_r) of an operand (componentwise, rounded to
// the nearest integer, ties to even: step 3) and every 2M modulus m_l with
// root s_l, the kernel writes the two int8 residues
//     A+ = (x_re + s x_im) mod m,   A- = (x_re - s x_im) mod m      (eq. 2m-pre)
// in the symmetric range [-(m-1)/2, (m-1)/2] into the operand planes 2l and
// 2l+1, in the fragment order the int8 GEMM consumes (o2m_internal.h).  For
// the 3M moduli of a hybrid set it writes x_re, x_im and x_re + x_im mod m
// into three planes (3M after reduction, Section 3.2); for even m = 256 the
// low byte of the residue in [-128, 128] is the int8 residue (-128 = 128).
//
// Exact residues without integer division: x (an integer held exactly in a
// double) is split into D base-2^26 digits x = sum_d x_d 2^(26 d), peeled
// from the top so that |x_d| <= 2^25 below the top digit; then
// R = sum_d c_d x_d = x (mod m) with c_d = 2^(26 d) mod m (symmetric),
// likewise I for x_im.  The host picks D from the bound on |x| so that the top
// digit stays below 2^36 (D = 2 up to 2^62, 3 up to 2^88; D = 4, 5 keep it
// below 2^30 and hold the digits as int32), which keeps |R| < 2^43.01 and
// A+- = R +- s I an exact integer below 2^51 (s <= 120).  Up to |x| <= 2^44
// no split is needed (D = 1: R = x, and |A+-| <= 121 2^44 < 2^51).  q = rint(A / m)
// comes out of one fma against 1.5 2^52 (the low word of the sum is q), and
// A - q m, needed only modulo 2^8, is one 24-bit integer multiply-add on the
// low words.
//
// Bound: HBM.  Algorithmic bytes per complex fp64 input element:
// 16 read + 2N written (8 + 2N for fp32 input).
#include "o2m_internal.h"

#include <string.h>
#include <type_traits>

namespace o2m {
namespace {

constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52

// Digit storage: exact doubles for D <= 3, int32 for D >= 4 (digits < 2^30).
template <int D> struct Digit { typedef double type; };
template <> struct Digit<4> { typedef int type; };
template <> struct Digit<5> { typedef int type; };

// x = sum_d dg[d] 2^(26 d), peeled from the top digit down (each step exact).
template <int D, int PT, typename DT>
__device__ inline void split_digits(double x, DT (&dg)[D][PT], int e) {
#pragma unroll
    for (int d = D - 1; d >= 1; --d) {
        const double q = rint(ldexp(x, -26 * d));
        x = fma(-q, ldexp(1.0, 26 * d), x);
        dg[d][e] = (DT)q;
    }
    dg[0][e] = (DT)x;
}

template <ElemType ET> struct Load;
template <> struct Load<kF64> {
    static __device__ inline double2 get(const void *X, size_t idx) {
        return reinterpret_cast<const double2 *>(X)[idx];
    }
};
template <> struct Load<kF32> {
    static __device__ inline double2 get(const void *X, size_t idx) {
        const float2 v = reinterpret_cast<const float2 *>(X)[idx];
        return make_double2((double)v.x, (double)v.y);
    }
};
template <> struct Load<kR64> {
    static __device__ inline double2 get(const void *X, size_t idx) {
        return make_double2(reinterpret_cast<const double *>(X)[idx], 0.0);
    }
};
template <> struct Load<kI32> {
    static __device__ inline double2 get(const void *X, size_t idx) {
        const int2 v = reinterpret_cast<const int2 *>(X)[idx];
        return make_double2((double)v.x, (double)v.y);
    }
};

__device__ inline uint32_t lo32(double d) { return (uint32_t)__double2loint(d); }

// a * b + c on the low 24 bits of a and b (v_mad_u32_u24)
__device__ inline uint32_t mad24(uint32_t a, uint32_t b, uint32_t c) { return __umul24(a, b) + c; }

__device__ inline uint32_t pack4(uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3) {
    const uint32_t lo = __builtin_amdgcn_perm(b1, b0, 0x0c0c0400u);  // [b0.0, b1.0, 0, 0]
    const uint32_t hi = __builtin_amdgcn_perm(b3, b2, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);                // [lo.0, lo.1, hi.0, hi.1]
}

// k entries per thread: one lane chunk of a fragment (16) for one digit, half
// of one from two digits on, a fragment then going to two waves, 32 chunks
// each.  With 16 entries the digits take 128 registers and more (two digits:
// three waves per SIMD instead of four, three: two instead of four, four and
// five: one), and the last round of waves costs more: residue phase at two
// digits 2048^3 75 -> 68 us, 500 x 333 x 777 15.9 -> 13.3, 4096 x 96 x 4096
// 159 -> 155, 8192^3 level; three digits 3000^3 N = 20 239 -> 221.  With one
// digit (fp32 operands) 16 entries read whole lines with fewer loads: 8 took
// 36 us instead of 30 for CGEMM 1537 x 1283 x 2051.
// The split form loads two real entries for one (SYRK, DSYR2K), and 16 of those
// spilled 24 registers: 8 as well (DSYRK 1200 x 3400 N = 10 20.6 -> 17.2 us, 800 x
// 2400 14.4 -> 12.2, 4096^2 N = 4 46.7 -> 44.3, 3000 x 5000 N = 10 53.3 -> 51.2).
template <int D, bool SPLIT> constexpr int per_thread() { return D == 1 && !SPLIT ? 16 : 8; }

// The split of the moduli (mchunk): waves that a launch is brought to, and
// moduli that a wave keeps at least.  2048 waves are two per SIMD; below, the
// serial chain of a wave is what takes the time (500 x 333 x 777, 1456 waves:
// residue phase 14.1 us whole, 13.0 in two parts, 13.9 in four, 16.3 in eight;
// 96 x 80 x 200, 160 waves: 12.1 whole, 7.5 in eight), above, the entries read
// again cost more than the split gives (700^3, 2112 waves: 14.8 whole, 15.7 in
// two parts).  With one digit and 16 entries per lane a wave does twice the
// work of a launch of twice as many, and registers hold three to a SIMD: 768
// (residue phase whole and in two parts: ZHERK 1088 x 1600 N = 10, 1700 waves,
// 15.6 and 21.4 us, 600 x 1200, 722 waves, 11.4 and 11.5, in four 14.0; ZGEMM
// 600 x 600 x 1300 N = 10, 1596 waves, 16.1 and 19.0; Gauss 666 x 666 x 1400
// 10.4 and 12.5; ZHERK 500 x 1000, 512 waves, 12.4 whole, 10.2 in two parts, 11.1
// in four).
constexpr long kResidueWaves = 2048, kResidueWavesWhole = 768;
constexpr int kMinModuli = 2;

// PT residue bytes of one lane, contiguous in the plane (16- or 8-byte store).
// The stores are non-temporal (no cache allocation): the planes are far
// larger than the caches and are read back only by the GEMM, from its own
// tile windows; plain stores measured 4-5% slower for the whole pass.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
template <int PT>
__device__ inline void store_words(int8_t *dst, const uint32_t (&w)[PT / 4]) {
    if constexpr (PT == 16) {
        const u32x4 v = {w[0], w[1], w[2], w[3]};
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
    } else {
        const u32x2 v = {w[0], w[1]};
        __builtin_nontemporal_store(v, reinterpret_cast<u32x2 *>(dst));
    }
}

// One launch takes up to two sources (the A and the B operand of a GEMM, the
// two matrices of a rank-2k update): its workgroups are the first source's,
// then the second's.  Two launches left the chip draining twice: residue phase
// at N = 16, two launches -> one, 1024^3 37 -> 25 us, 2048^3 88 -> 76 us,
// 96 x 80 x 200 33 -> 9 us (there mostly the loads at the edges, which went out
// one at a time, and the split of the moduli), 8192^3 level.  Per source (ResidueSource, o2m_internal.h):
//   rows (mode 0): operand rows are rows of X, entry (r, kk) at X[r + kk*ld]
//   columns (mode 1): operand rows are columns of X, (r, kk) at X[kk + r*ld]
//   SPLIT (SYRK, rows only): X real, (r, kk) = X[r + kk ld] + i X[r + (kk+kh) ld]
//   conj: the operand is the complex conjugate of X (imaginary parts negated)
// D: base-2^26 digits of the quantized values (1..5, from their bound)
// PAIRS (complex fp32, the host sets it when every pair is 16-byte aligned):
// columns read two consecutive entries per 16-byte load; rows read rows 2i,
// 2i + 1 of a column per 16-byte load, the lane of the even row the first half
// of its columns and the lane of the odd row the second, and the two then swap
// so that each lane holds its own row's entries
//
// Workgroup row blockIdx.y computes the moduli [y mchunk, (y + 1) mchunk): a
// wave's 2N residues per entry are a serial chain of ~100 instructions per
// entry, so an operand of few fragments left most of the chip idle behind
// them (1024 x 1024: one wave per SIMD).  Splitting the moduli re-reads the
// entries, from the caches at those sizes (launch_residues).
struct ResidueArgs {
    ResidueSource src[2];
    unsigned blocks0;        // workgroups of src[0]
    int mchunk;
    ResidueParams rp;
};

template <ElemType ET, int D, bool SCALED, bool PAIRS, bool SPLIT>
__global__ __launch_bounds__(256, D == 1 ? 3 : 1) void residue_kernel(ResidueArgs a) {
    constexpr int PT = per_thread<D, SPLIT>();
    constexpr int kHalves = 16 / PT;                          // waves per fragment
    const ResidueParams &rp = a.rp;
    // what the loads need is read of both sources at once and then selected:
    // a read of the selected source would wait for the selection first
    const ResidueSource &s0 = a.src[0], &s1 = a.src[1];
    asm volatile("" ::"s"(a.blocks0), "s"(s0.X), "s"(s1.X), "s"(s0.E), "s"(s1.E), "s"(s0.ld), "s"(s1.ld),
                 "s"(s0.g.rows), "s"(s1.g.rows), "s"(s0.g.k), "s"(s1.g.k), "s"(s0.g.rows_pad), "s"(s1.g.rows_pad),
                 "s"(s0.g.kblocks), "s"(s1.g.kblocks), "s"(s0.mode), "s"(s1.mode));
    const bool second = blockIdx.x >= a.blocks0;
    const ResidueSource &o = second ? s1 : s0;   // what is used later
    const unsigned block = blockIdx.x - (second ? a.blocks0 : 0u);
    const bool cols = !SPLIT && (second ? s1.mode : s0.mode) == 1;
    const void *X = second ? s1.X : s0.X;
    const int32_t *E = second ? s1.E : s0.E;
    const int rows = second ? s1.g.rows : s0.g.rows, k = second ? s1.g.k : s0.g.k, ld = second ? s1.ld : s0.ld;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(block * 4 + (threadIdx.x >> 6));  // wave-uniform
    const int frag = wave / kHalves, half = wave % kHalves;   // one fragment per kHalves waves
    const int frows = (second ? s1.g.rows_pad : s0.g.rows_pad) / kFragRows;  // fragments along rows
    const int fks = second ? s1.g.kblocks : s0.g.kblocks;                    // fragments along k
    if (frag >= frows * fks) return;
    // columns: walk k fastest (contiguous); rows: walk rows fastest
    const int per = cols ? fks : frows;
    const int hi = frag / per, lo = frag - hi * per;
    const int fk = cols ? lo : hi, fr = cols ? hi : lo;
    // the fragment's 16-byte lane chunk and the part of it this lane fills;
    // with two waves per fragment each takes 32 whole chunks (adjacent lanes
    // fill the two halves of one), so that a store covers 512 contiguous bytes
    const int chunk = kHalves == 1 ? lane : half * 32 + (lane >> 1);
    const int part = kHalves == 1 ? 0 : lane & 1;
    const int r = fr * kFragRows + (chunk & 15);
    const int kk0 = fk * kStageK + (chunk >> 4) * 16 + part * PT;

    // ---- load and quantize (step 3) -------------------------------------
    // Every load is taken unguarded, so that all of them are in flight before
    // the first is used.  (With a per-lane guard around each load the compiler
    // moves the quantization of the value into the guarded branch, where it
    // must wait for that load: the loads then go out one at a time.)  A wave
    // whose fragment (16 rows x 64 k) lies inside the operand reads it as it
    // is; at the edges the indices are clamped into the operand and the values
    // beyond it dropped.
    typedef typename Digit<D>::type DT;
    DT xr[D][PT], xi[D][PT];
    const bool inner = fr * kFragRows + kFragRows <= rows && fk * kStageK + kStageK <= k &&
                       (!SPLIT || fk * kStageK + kStageK + o.khalf <= o.g.kreal);
    // the row's exponent is fetched first and used once the entries' loads
    // are issued (every padded row has an entry)
    int erow = 0;
    if constexpr (SCALED) erow = E[r];
    int sh = 0;
    bool live = r < rows;                    // bounds only until settle()
    auto settle = [&]() {
        if constexpr (SCALED) {
            live = live && erow != INT32_MIN;  // non-finite row: output masked later
            sh = o.shift - erow;
        }
    };
    auto put = [&](int e, double vr, double vi) {
        if (!live) vr = vi = 0.0;
        if (o.g.conj) vi = -vi;              // conjugated operand: exact
        if (SCALED) {
            vr = rint(ldexp(vr, sh));
            vi = rint(ldexp(vi, sh));
        }
        split_digits<D, PT>(vr, xr, e);
        split_digits<D, PT>(vi, xi, e);
    };
    auto load_single = [&](auto edge, auto columns) {
        constexpr bool EDGE = decltype(edge)::value, COLS = decltype(columns)::value;
        // entry (rc, kc) at index base + kc ks
        const int rc = EDGE ? min(r, rows - 1) : r;
        const size_t ks = COLS ? 1 : (size_t)ld;
        const size_t base = COLS ? (size_t)rc * ld : (size_t)rc;
        const size_t first = base + kk0 * ks;
        double vr[PT], vi[PT];
#pragma unroll
        for (int e = 0; e < PT; ++e) {
            const size_t at = EDGE ? base + min(kk0 + e, k - 1) * ks : first + e * ks;
            if constexpr (!SPLIT) {
                const double2 v = Load<ET>::get(X, at);
                vr[e] = v.x; vi[e] = v.y;
            } else {
                const double *Xr = reinterpret_cast<const double *>(X);
                vr[e] = Xr[at];
                vi[e] = Xr[EDGE ? base + min(kk0 + e + o.khalf, o.g.kreal - 1) * ks : at + o.khalf * ks];
            }
        }
        settle();
#pragma unroll
        for (int e = 0; e < PT; ++e) {
            if (EDGE && kk0 + e >= k) vr[e] = vi[e] = 0.0;
            if (EDGE && SPLIT && kk0 + e + o.khalf >= o.g.kreal) vi[e] = 0.0;
            put(e, vr[e], vi[e]);
        }
    };
    auto load_pairs = [&]() {
        const float2 *Xf = reinterpret_cast<const float2 *>(X);
        if (cols) {
            const float2 *Xc = Xf + (size_t)r * ld + kk0;
            float4 v[PT / 2];
#pragma unroll
            for (int e = 0; e < PT / 2; ++e) v[e] = *reinterpret_cast<const float4 *>(Xc + 2 * e);
            settle();
#pragma unroll
            for (int e = 0; e < PT / 2; ++e) {
                put(2 * e, (double)v[e].x, (double)v[e].y);
                put(2 * e + 1, (double)v[e].z, (double)v[e].w);
            }
        } else {
            constexpr int kPair = kHalves;          // lanes between a row and its pair's other row
            const bool odd = lane & kPair;
            const float2 *Xa = Xf + (r - (int)odd) + (size_t)(kk0 + (odd ? PT / 2 : 0)) * ld;   // the pair's even row
            float4 v[PT / 2];
#pragma unroll
            for (int j = 0; j < PT / 2; ++j) v[j] = *reinterpret_cast<const float4 *>(Xa + (size_t)j * ld);
            settle();
#pragma unroll
            for (int j = 0; j < PT / 2; ++j) {
                // the even lane passes on its odd row's half, the odd lane its even row's
                const float rx = __shfl_xor(odd ? v[j].x : v[j].z, kPair, 64);
                const float ry = __shfl_xor(odd ? v[j].y : v[j].w, kPair, 64);
                put(j, odd ? rx : v[j].x, odd ? ry : v[j].y);
                put(PT / 2 + j, odd ? v[j].z : rx, odd ? v[j].w : ry);
            }
        }
    };
    // a fragment of padding only has nothing to read: zero residues
    const bool padding = fr * kFragRows >= rows || fk * kStageK >= k;
    if (__builtin_expect(inner, 1)) {
        if constexpr (PAIRS) load_pairs();
        else if (!SPLIT && cols) load_single(std::false_type(), std::true_type());
        else load_single(std::false_type(), std::false_type());
    } else if (!padding) {
        if (!SPLIT && cols) load_single(std::true_type(), std::true_type());
        else load_single(std::true_type(), std::false_type());
    }

    const size_t plane_bytes = o.g.plane_bytes;
    int8_t *dst_p = o.planes + plane_offset(r, kk0 + o.g.kofs_p * kStageK, o.g.plane_kblocks);
    int8_t *dst_m = o.planes + plane_offset(r, kk0 + o.g.kofs_m * kStageK, o.g.plane_kblocks) + plane_bytes;
    const int l0 = blockIdx.y * a.mchunk, l1 = min(rp.n, l0 + a.mchunk);
    const int l2m = min(rp.n2, l1), l3m = max(rp.n2, l0);   // 2M moduli [l0, l2m), 3M [l3m, l1)
    if (padding) {
        const uint32_t z[PT / 4] = {};
        for (int l = l0; l < l2m; ++l) {
            store_words<PT>(dst_p + (size_t)(2 * l) * plane_bytes, z);
            store_words<PT>(dst_m + (size_t)(2 * l) * plane_bytes, z);
        }
        for (int l = l3m; l < l1; ++l)
            for (int c = 0; c < 3; ++c)
                store_words<PT>(dst_p + (size_t)(2 * rp.n2 + 3 * (l - rp.n2) + c) * plane_bytes, z);
        return;
    }

    // ---- residues and 2M pre per modulus (step 4, eq. 2m-pre) -------------
    for (int l = l0; l < l2m; ++l) {
        const double inv = rp.inv[l];
        const double s = (double)rp.root[l];
        const uint32_t negm = (uint32_t)(-rp.mod[l]) & 0xFFFFFFu;
        uint32_t wp[PT / 4], wm[PT / 4];
#pragma unroll
        for (int q = 0; q < PT / 4; ++q) {
            uint32_t bp[4], bm[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int e = 4 * q + t;
                double R = (double)xr[0][e], I = (double)xi[0][e];
#pragma unroll
                for (int d = 1; d < D; ++d) {
                    R = fma(rp.cpow[l][d - 1], (double)xr[d][e], R);
                    I = fma(rp.cpow[l][d - 1], (double)xi[d][e], I);
                }
                const double Ap = fma(s, I, R), Am = fma(-s, I, R);
                const double tp = fma(Ap, inv, kMagic), tm = fma(Am, inv, kMagic);
                const uint32_t ap = lo32(Ap + kMagic), am = lo32(Am + kMagic);
                bp[t] = mad24(lo32(tp), negm, ap);   // A+ - q m (low byte)
                bm[t] = mad24(lo32(tm), negm, am);
            }
            wp[q] = pack4(bp[0], bp[1], bp[2], bp[3]);
            wm[q] = pack4(bm[0], bm[1], bm[2], bm[3]);
        }
        store_words<PT>(dst_p + (size_t)(2 * l) * plane_bytes, wp);
        store_words<PT>(dst_m + (size_t)(2 * l) * plane_bytes, wm);
    }

    // ---- hybrid sets: residues of Xr, Xi and Xr + Xi for 3M (Section 3.2) ---
    for (int l = l3m; l < l1; ++l) {
        const double inv = rp.inv[l];
        const uint32_t negm = (uint32_t)(-rp.mod[l]) & 0xFFFFFFu;
        uint32_t w[3][PT / 4];
#pragma unroll
        for (int q = 0; q < PT / 4; ++q) {
            uint32_t by[3][4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int e = 4 * q + t;
                double R = (double)xr[0][e], I = (double)xi[0][e];
#pragma unroll
                for (int d = 1; d < D; ++d) {
                    R = fma(rp.cpow[l][d - 1], (double)xr[d][e], R);
                    I = fma(rp.cpow[l][d - 1], (double)xi[d][e], I);
                }
                const double v[3] = {R, I, R + I};
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double tq = fma(v[c], inv, kMagic);
                    by[c][t] = mad24(lo32(tq), negm, lo32(v[c] + kMagic));
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) w[c][q] = pack4(by[c][0], by[c][1], by[c][2], by[c][3]);
        }
        const size_t p0 = (size_t)(2 * rp.n2 + 3 * (l - rp.n2));
#pragma unroll
        for (int c = 0; c < 3; ++c)
            store_words<PT>(dst_p + (p0 + c) * plane_bytes, w[c]);
    }
}

}  // namespace

static bool pairs_of(ElemType et, const ResidueSource &s) {
    // complex fp32 entries in 16-byte pairs when every pair is aligned: along
    // a column (k-chunks start at even k) or across rows 2i, 2i + 1; an even
    // ld and a 16-byte aligned base suffice
    return et == kF32 && s.ld % 2 == 0 && ((uintptr_t)s.X & 15) == 0;
}

hipError_t launch_residues(ElemType et, bool split, int count, const ResidueSource *src, const ResidueParams &rp,
                           hipStream_t st) {
    if (count < 1 || count > 2) return hipErrorInvalidValue;
    const int digits = src[0].digits;
    const bool pairs = pairs_of(et, src[0]);
    if (count == 2 && (src[1].digits != digits || pairs_of(et, src[1]) != pairs)) {
        const hipError_t e = launch_residues(et, split, 1, src, rp, st);
        return e != hipSuccess ? e : launch_residues(et, split, 1, src + 1, rp, st);
    }
    // waves: one per fragment of 16 entries a lane, two of 8 (per_thread)
    const bool whole = digits == 1 && !split;
    long waves[2] = {0, 0};
    for (int i = 0; i < count; ++i)
        waves[i] = (long)(src[i].g.rows_pad / kFragRows) * (long)src[i].g.kblocks * (whole ? 1 : 2);
    const long blocks = (waves[0] + 3) / 4 + (waves[1] + 3) / 4;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    ResidueArgs a;
    memset(&a, 0, sizeof a);
    for (int i = 0; i < count; ++i) a.src[i] = src[i];
    a.blocks0 = (unsigned)((waves[0] + 3) / 4);
    // moduli per workgroup: split until the launch has that many waves
    const long target = digits == 1 ? kResidueWavesWhole : kResidueWaves;
    a.mchunk = rp.n;
    while (a.mchunk > kMinModuli && blocks * 4 * ((rp.n + a.mchunk - 1) / a.mchunk) < target)
        a.mchunk = (a.mchunk + 1) / 2;
    a.rp = rp;
    const dim3 grid((unsigned)blocks, (unsigned)((rp.n + a.mchunk - 1) / a.mchunk));
#define O2M_RES(T, DD, SC, PR, SP) residue_kernel<T, DD, SC, PR, SP><<<grid, 256, 0, st>>>(a)
#define O2M_RES_D(T, PR, SP)                               \
    switch (digits) {                                      \
    case 1: O2M_RES(T, 1, true, PR, SP); break;            \
    case 2: O2M_RES(T, 2, true, PR, SP); break;            \
    case 3: O2M_RES(T, 3, true, PR, SP); break;            \
    case 4: O2M_RES(T, 4, true, PR, SP); break;            \
    case 5: O2M_RES(T, 5, true, PR, SP); break;            \
    default: return hipErrorInvalidValue;                  \
    }
    if (split && et == kR64) { O2M_RES_D(kR64, false, true) }
    else if (split) return hipErrorInvalidValue;
    else if (et == kF64) { O2M_RES_D(kF64, false, false) }
    else if (et == kF32 && pairs) { O2M_RES_D(kF32, true, false) }
    else if (et == kF32) { O2M_RES_D(kF32, false, false) }
    else if (et == kI32) O2M_RES(kI32, 1, false, false, false);
    else return hipErrorInvalidValue;
#undef O2M_RES_D
#undef O2M_RES
    return hipGetLastError();
}

}  // namespace o2m
