// Device-side modular arithmetic for primes below 2^36, carried in IEEE double precision.
//
// gfx950 issues double-precision FMA, multiply, add and round at the rate of a 32-bit integer multiply
// (measured, four wavefronts per SIMD, cycles per wavefront instruction: fma_f64 5.3, add_f64 5.2, mul_lo_u32
// and mul_hi_u32 4.9, mad_u64_u32 5.6), so a modular product of two 36-bit residues is six instructions as a
// Barrett reduction with an FMA-based exact product, against about a dozen 32-bit partial products and carries.  Every quantity below is an
// integer-valued double of magnitude < 2^53, hence exact; only the quotient estimate is approximate,
// and its error merely moves the result to another small representative of the same residue class.
//
// "Lazy" values: a residue may be held as any integer r with |r| <= 16 p congruent to the true
// value (Kernel Code Generation: lazy modular reduction); `canon` produces the canonical one.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// The arithmetic is plain IEEE double arithmetic, so it is callable from host code as well; the CPU-only test
// suite uses that to check every bound stated below against 128-bit integer arithmetic.
#define KS_HD __host__ __device__ __forceinline__

namespace ks {

struct Mod {
    double p;     // the modulus
    double pinv;  // 1/p rounded to nearest
};

constexpr double kTwo52 = 4503599627370496.0;

// Exact for x < 2^52: plant x in the mantissa of 2^52 and subtract 2^52.
KS_HD double u64_to_f64(uint64_t x) {
    return __builtin_bit_cast(double, x | 0x4330000000000000ull) - kTwo52;
}
// Exact for integer-valued 0 <= r < 2^52.
KS_HD uint64_t f64_to_u64(double r) {
    return __builtin_bit_cast(uint64_t, r + kTwo52) & 0x000FFFFFFFFFFFFFull;
}

// Residues at the library boundary are stored in 64-bit words or, for moduli below 2^32, in 32-bit words.
template <typename W>
KS_HD double word_to_f64(W x);
template <>
KS_HD double word_to_f64<uint64_t>(uint64_t x) { return u64_to_f64(x); }
template <>
KS_HD double word_to_f64<uint32_t>(uint32_t x) { return (double)x; }
template <typename W>
KS_HD W f64_to_word(double r);  // integer-valued canonical residue
template <>
KS_HD uint64_t f64_to_word<uint64_t>(double r) { return f64_to_u64(r); }
template <>
KS_HD uint32_t f64_to_word<uint32_t>(double r) { return (uint32_t)r; }

// a * b mod p as a small signed representative.
// Requires integer-valued |a| <= 2^43, |b| <= 2^36.  Returns r = a b (mod p) with |r| <= 0.51 p.
//   h + l = a b exactly (l is the rounding error of the product, recovered by one FMA);
//   q ~ a b / p; h - q p is an integer below 2^36 in magnitude, so the second FMA is exact too.
KS_HD double mulmod_lazy(double a, double b, Mod m) {
    double h = a * b;
    double l = __builtin_fma(a, b, -h);
    double q = __builtin_rint(h * m.pinv);
    double r = __builtin_fma(-q, m.p, h);
    return r + l;
}

// Any integer-valued |x| < 2^53 -> representative with |r| <= 0.51 p (the quotient estimate is off by at most one
// part in 2^51, the FMA is exact because its result is).
KS_HD double reduce_lazy(double x, Mod m) {
    double q = __builtin_rint(x * m.pinv);
    return __builtin_fma(-q, m.p, x);
}

// Exact multiply-accumulate of residues: (hi - kMacBias) + lo is the running sum of products as an integer.  hi lives in
// [2^80, 2^81), where doubles are 2^28 apart, so fma(x, k, hi) rounds x k to a multiple of 2^28; the part it dropped,
// x k - (hi_new - hi), is an integer of magnitude <= 2^27 that the second FMA recovers exactly and lo collects.  Four
// instructions a product and one reduction per sum, where a Barrett product and an addition take seven.
// Requires |x|, |k| <= 2^36 and sums of at most 2^79: kMacTerms products, or kMacTermsLazy if |k| <= 0.51 * 2^36 (a lazy
// residue; 0.51 * 250 < 128).
constexpr double kMacBias = 0x1.8p80;
constexpr int kMacTerms = 128, kMacTermsLazy = 250;
KS_HD void mac_exact(double x, double k, double& hi, double& lo) {
    const double t = __builtin_fma(x, k, hi);
    const double d = hi - t;
    lo += __builtin_fma(x, k, d);
    hi = t;
}
// The sum of a mac_exact accumulation as a lazy residue (|r| <= 0.51 p).  With |x| <= 2^36 and |k| <= p the quotient
// of the high part stays below 2^44 whatever p is, so its estimate is off by far less than one and the FMA is exact.
KS_HD double mac_reduce(double hi, double lo, Mod m) {
    const double s = hi - kMacBias;
    const double q = __builtin_rint(s * m.pinv);
    return reduce_lazy(__builtin_fma(-q, m.p, s) + lo, m);
}

// The same in two instructions where the low words of both factors are at hand as integers: hi is the sum of the products in doubles,
// rounded at each step, and the low 32 bits of lo are the exact sum modulo 2^32, which tell by how much hi is off as long as that is less
// than 2^31.  Requires |x| <= 2^36 (a residue, or a sum that mac_wide_reduce left: 0.51 p + 2^31, which may be more than p) and |k| <= p.  The sum
// of T products then stays below T 2^36 p <= T 2^72 and the roundings below T^2 2^19: T <= kMacWideTerms.
constexpr int kMacWideTerms = 60;
KS_HD void mac_wide(double x, double k, uint32_t x_low, uint32_t k_low, double& hi, uint64_t& lo) {
    hi = __builtin_fma(x, k, hi);
    lo += (uint64_t)x_low * k_low;
}
// The sum as a representative |r| <= 0.51 p + 2^31, and its low word.
KS_HD double mac_wide_reduce(double hi, uint64_t lo, Mod m, uint32_t* low) {
    constexpr double kRound = 6755399441055744.0;   // 1.5 * 2^52: the low word of x + kRound is that of the integer x, |x| < 2^51
    const double q = __builtin_rint(hi * m.pinv), r = __builtin_fma(-q, m.p, hi);   // |q| <= T 2^36 < 2^42; r is an integer below 2^36: exact
    const uint32_t q_low = (uint32_t)__builtin_bit_cast(uint64_t, q + kRound), r_low = (uint32_t)__builtin_bit_cast(uint64_t, r + kRound);
    const uint32_t p_low = (uint32_t)__builtin_bit_cast(uint64_t, m.p + kRound);
    const int32_t off = (int32_t)((uint32_t)lo - r_low - q_low * p_low);
    *low = r_low + (uint32_t)off;
    return r + (double)off;
}

// The same for moduli below 2^28: 64-bit integer multiply-adds, one instruction a product at the rate of a double-precision FMA.
// 0 <= x < p and |k| <= p, or |k| <= 0.51 p: kMacTerms or kMacTermsLazy products stay below 2^63, with a start below 2^28.
KS_HD void mac_int(int32_t x, int32_t k, int64_t& sum) { sum += (int64_t)x * k; }
// The high word times 2^32 and the low word are both exact doubles; the quotient is at most 250 p < 2^36 in magnitude.
KS_HD double mac_int_reduce(int64_t sum, Mod m) {
    const double s = (double)(int32_t)(sum >> 32) * 4294967296.0;
    const double q = __builtin_rint(s * m.pinv);
    return reduce_lazy(__builtin_fma(-q, m.p, s) + (double)(uint32_t)sum, m);
}

// Split an integer-valued |y| < 2^36 into y = y2 + y1 + y0 with y2 a multiple of 2^24 (|y2| <= 2^36), y1 a
// multiple of 2^12 (|y1| <= 2^23) and |y0| <= 2^11, by rounding to nearest at the two granularities (adding and
// subtracting 1.5 * 2^(52 + g) rounds to a multiple of 2^g).  Six additions, no products.
// Use: with factors f_k = centred([f * 2^(12 k)]_t) * 2^(-12 k), |f_k| * 2^(12 k) <= 2^35, the sum
// y2 f_2 + y1 f_1 + y0 f_0 is an integer congruent to y f modulo t and at most 2^48 in magnitude, so up to seventeen
// such triples accumulate exactly in one double: a conversion costs three FMAs per source and target, the split is
// shared by all targets of the source, and one reduction per target finishes it.
KS_HD void split3(double y, double& y2, double& y1, double& y0) {
    constexpr double kRound24 = 0x1.8p76, kRound12 = 0x1.8p64;
    y2 = (y + kRound24) - kRound24;
    const double rem = y - y2;
    y1 = (rem + kRound12) - kRound12;
    y0 = rem - y1;
}

// The same for |y| < 2^32 (contexts whose moduli are all below 2^32, i.e. every context the 32-bit-word entry points
// accept, the paper's 28-bit primes included): y = y1 + y0 with y1 a multiple of 2^16 and |y0| <= 2^15.  With
// f_k = centred([f * 2^(16 k)]_t) * 2^(-16 k), |f_k| * 2^(16 k) <= 2^31, the sum y1 f_1 + y0 f_0 is an integer congruent to
// y f modulo t and below 1.5 * 2^47 in magnitude: seventeen accumulate exactly (below 2^53), at two FMAs per source and
// target and three additions per split.
KS_HD void split2(double y, double& y1, double& y0) {
    constexpr double kRound16 = 0x1.8p68;
    y1 = (y + kRound16) - kRound16;
    y0 = y - y1;
}

// The fused conversion takes the 40 bits of y + 0x80808080 (|y| < 2^36; low word w, signed byte `top`) apart as they lie in memory.
// Three pieces: the low 12 bits, the next 12 in place and what is left shifted down by 24, against f_0, f_1 as above and 2^24 f_2:
// products of at most 2^47, 2^47 and 2^47.1.  Two (|y| < 2^32): the low 16 bits and the rest, against f_0 and 2^16 f_1, 2^47 and
// 1.5 * 2^47.  Those of seventeen sources and a start below 2^35, which takes the constants out, stay below 2^52.8.
template <int PIECES>
KS_HD void cut_source(uint32_t w, int top, double (&p)[PIECES]) {
    static_assert(PIECES == 2 || PIECES == 3, "pieces of a source");
    const uint64_t bits = (uint64_t)(uint32_t)top << 32 | w;
    if constexpr (PIECES == 3) {
        p[0] = (double)(w & 0xFFFu);
        p[1] = (double)(w & 0xFFF000u);
        p[2] = (double)(int)(uint32_t)(bits >> 24);
    } else {
        p[0] = (double)(w & 0xFFFFu);
        p[1] = (double)(int)(uint32_t)(bits >> 16);
    }
}

// Representative in (-p, p) -> canonical [0, p).
KS_HD double canon(double r, Mod m) { return r < 0.0 ? r + m.p : r; }

// The 15 twiddles of a 16-point register pass: t[2^u + g] = W[(base << u) + g] for local stage u = 0..3 and
// group g < 2^u, i.e. the sub-tree below heap node `base` of the per-modulus table W[k] = psi^brv(k).
// Loading them ahead of the butterflies lets their latency overlap the data loads.
KS_HD void load_twiddles16(double (&t)[16], const double* __restrict__ W, uint32_t base) {
    t[0] = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int g = 0; g < (1 << u); ++g) t[(1 << u) + g] = W[(base << u) + g];
}

// Sixteen points, four decimation-in-time stages, in registers.  v[k] are 16 points whose mutual distances
// are 8, 4, 2, 1 times a common stride.  Growth: every stage adds at most 0.51 p to the magnitude.
// U0 > 0 runs only the local stages U0..3 (the last 4 - U0 stages: distances 8 >> U0 .. 1), for passes shorter than four
// stages; the table layout is the same.
template <int U0 = 0>
KS_HD void radix16_fwd(double (&v)[16], const double (&t)[16], Mod m) {
#pragma unroll
    for (int u = U0; u < 4; ++u) {
        const int half = 8 >> u;
#pragma unroll
        for (int g = 0; g < (1 << u); ++g) {
            const double w = t[(1 << u) + g];
#pragma unroll
            for (int i = 0; i < half; ++i) {
                const int k = g * 2 * half + i;
                const double x = mulmod_lazy(v[k + half], w, m);
                v[k + half] = v[k] - x;
                v[k] = v[k] + x;
            }
        }
    }
}

// Inverse of radix16_fwd up to the factor 16 (decimation in frequency) with t built from Winv[k] = psi^-brv(k).
// Inputs must satisfy |v| <= p; sums double per stage, so outputs are bounded by 16 p.
template <int U0 = 0>
KS_HD void radix16_inv(double (&v)[16], const double (&t)[16], Mod m) {
#pragma unroll
    for (int u = 3; u >= U0; --u) {
        const int half = 8 >> u;
#pragma unroll
        for (int g = 0; g < (1 << u); ++g) {
            const double w = t[(1 << u) + g];
#pragma unroll
            for (int i = 0; i < half; ++i) {
                const int k = g * 2 * half + i;
                const double x = v[k], y = v[k + half];
                v[k] = x + y;
                v[k + half] = mulmod_lazy(x - y, w, m);
            }
        }
    }
}

}  // namespace ks
