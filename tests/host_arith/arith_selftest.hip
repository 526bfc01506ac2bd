// Host-side check of the library's double-precision modular arithmetic (ks_device.hpp) against exact
// 128-bit integer arithmetic, and of the conversion tables that the built library makes.  Runs entirely on the CPU; prints "OK" and exits 0 when every bound holds.
#include <stdio.h>
#include <stdlib.h>
#include <math.h>
#include <stdint.h>
#include <string.h>
#include <vector>
#include "../../paper_2512_11269_amd/csrc/ks_internal.hpp"
#include "../../paper_2512_11269_amd/csrc/ks_tiles.hpp"

using namespace ks;
typedef __int128 i128;

static uint64_t rng_state = 0x9E3779B97F4A7C15ull;
static uint64_t rnd() {  // xorshift64*
    rng_state ^= rng_state >> 12; rng_state ^= rng_state << 25; rng_state ^= rng_state >> 27;
    return rng_state * 0x2545F4914F6CDD1Dull;
}
static int64_t rnd_signed(int bits) { return (int64_t)(rnd() >> (64 - bits)) - ((int64_t)1 << (bits - 1)); }
static int fails = 0;
#define CHECK(cond, ...) do { if (!(cond)) { if (fails < 20) { printf("FAIL %s:%d: ", __FILE__, __LINE__); printf(__VA_ARGS__); printf("\n"); } ++fails; } } while (0)

static int64_t mod_i128(i128 x, int64_t p) { i128 r = x % p; if (r < 0) r += p; return (int64_t)r; }

static void check_prime(uint64_t p) {
    const Mod m{(double)p, 1.0 / (double)p};
    const double lim = 0.51 * (double)p;
    // conversions
    for (int i = 0; i < 20000; ++i) {
        uint64_t x = rnd() >> 12;
        if (i < 4) x = (uint64_t[]){0, 1, p - 1, (1ull << 52) - 1}[i];
        CHECK(u64_to_f64(x) == (double)x, "u64_to_f64 %llu", (unsigned long long)x);
        CHECK(f64_to_u64((double)x) == x, "f64_to_u64 %llu", (unsigned long long)x);
    }
    // mulmod_lazy: |a| <= 2^43, 0 <= b < p (also negative b up to p in magnitude)
    for (int i = 0; i < 400000; ++i) {
        int64_t a = rnd_signed(44), b = (int64_t)(rnd() % p);
        if (i % 7 == 0) a = (i & 8) ? ((int64_t)1 << 43) : -((int64_t)1 << 43);
        if (i % 11 == 0) b = (int64_t)p - 1;
        if (i % 13 == 0) { int64_t k = rnd_signed(40); i128 t = (i128)k * p + rnd_signed(3); b = 1; a = (int64_t)t; if (a > ((int64_t)1 << 43) || a < -((int64_t)1 << 43)) a = k; }
        if (i % 17 == 0) b = -b;
        const double r = mulmod_lazy((double)a, (double)b, m);
        CHECK(r == floor(r), "mulmod not integer");
        CHECK(fabs(r) <= lim, "mulmod bound a=%lld b=%lld r=%.0f p=%llu", (long long)a, (long long)b, r, (unsigned long long)p);
        CHECK(mod_i128((i128)(int64_t)r, p) == mod_i128((i128)a * b, p), "mulmod value a=%lld b=%lld", (long long)a, (long long)b);
        const double c = canon(r, m);
        CHECK(c >= 0 && c < (double)p && (int64_t)c == mod_i128((i128)a * b, p), "canon");
    }
    // products that land exactly on / next to multiples of p and half-multiples (rounding boundaries of the quotient)
    for (int i = 0; i < 100000; ++i) {
        const int64_t b = (int64_t)(rnd() % (p - 1)) + 1;
        const int64_t q = (int64_t)(rnd() >> 24);
        i128 target = (i128)q * p + ((i & 1) ? (i128)(p / 2) : 0) + rnd_signed(3);
        int64_t a = (int64_t)(target / b);
        if (a > ((int64_t)1 << 43) || a < -((int64_t)1 << 43)) continue;
        const double r = mulmod_lazy((double)a, (double)b, m);
        CHECK(fabs(r) <= lim && mod_i128((i128)(int64_t)r, p) == mod_i128((i128)a * b, p), "mulmod boundary a=%lld b=%lld", (long long)a, (long long)b);
    }
    // reduce_lazy: any |x| < 2^53
    for (int i = 0; i < 200000; ++i) {
        int64_t x = rnd_signed(54);
        if (i % 5 == 0) x = (int64_t)((rnd() >> 40) * p) + rnd_signed(3) + ((i & 1) ? (int64_t)(p / 2) : 0);
        if (x >= ((int64_t)1 << 53) || x <= -((int64_t)1 << 53)) continue;
        const double r = reduce_lazy((double)x, m);
        CHECK(fabs(r) <= lim && mod_i128((i128)(int64_t)r, p) == mod_i128((i128)x, p), "reduce x=%lld r=%.0f", (long long)x, r);
    }
    // mac_exact: as many products as it takes, of the largest operands and of smaller ones, reduced once; the high sum stays
    // where doubles are 2^28 apart
    for (int rep = 0; rep < 3000; ++rep) {
        double hi = kMacBias, lo = 0.0;
        i128 exact = 0;
        const int terms = rep % 3 == 0 ? kMacTermsLazy : kMacTerms;
        for (int i = 0; i < terms; ++i) {
            int64_t x = (int64_t)(rnd() % p), k = (int64_t)(rnd() % p);
            if (rep % 5 == 0) x = p - 1;
            if (rep % 3 == 0) k = rep % 5 == 0 ? (int64_t)(0.51 * p) * (rep & 1 ? -1 : 1) : k / 2 - (int64_t)(p / 4);
            else if (rep % 5 == 0) k = p - 1;
            mac_exact((double)x, (double)k, hi, lo);
            exact += (i128)x * k;
            CHECK(hi >= 0x1p80 && hi < 0x1p81, "mac_exact high sum after %d of %d terms", i + 1, terms);
        }
        CHECK(lo == floor(lo) && fabs(lo) <= terms * 134217728.0, "mac_exact low sum");
        CHECK((i128)(hi - kMacBias) + (i128)(int64_t)lo == exact, "mac_exact sum");
        const double r = mac_reduce(hi, lo, m);
        CHECK(fabs(r) <= lim && mod_i128((i128)(int64_t)r, p) == mod_i128(exact, p), "mac_reduce");
    }
    // mac_wide: as many products as it takes, of the largest operands of one sign (the largest roundings) and of others, from a lazy start
    for (int rep = 0; rep < 3000; ++rep) {
        const int64_t start = rep % 3 == 0 ? 0 : rnd_signed(37);
        double hi = (double)start;
        uint64_t lo = (uint32_t)start;
        i128 exact = start;
        const double most = 68719476736.0;   // 2^36
        for (int i = 0; i < kMacWideTerms; ++i) {
            // the first factor is any of up to 2^36 (the reduced sum that it may be exceeds a small modulus), the second a residue
            const int64_t reduced = (int64_t)(0.51 * (double)p) + 2147483648ll;
            int64_t x = rep % 5 == 0 ? (int64_t)most - (int64_t)(rnd() & 0xFF) : rep % 5 == 1 ? rnd_signed(37) : rep % 5 == 2 ? (i & 1 ? -reduced : reduced) : (int64_t)(rnd() % p);
            int64_t k = rep % 7 == 0 ? (int64_t)p - (int64_t)(rnd() & 0xFF) : (int64_t)(rnd() % p);
            if (rep % 5 == 1 && (x > (int64_t)most || x < -(int64_t)most)) x /= 2;
            mac_wide((double)x, (double)k, (uint32_t)x, (uint32_t)k, hi, lo);
            exact += (i128)x * k;
        }
        uint32_t low;
        const double r = mac_wide_reduce(hi, lo, m, &low);
        CHECK(fabs(r) <= 0.51 * (double)p + 2147483648.0 && mod_i128((i128)(int64_t)r, p) == mod_i128(exact, p), "mac_wide_reduce");
        CHECK(low == (uint32_t)(int64_t)r, "mac_wide_reduce low word");
    }
    // mac_int (moduli below 2^28): the same with 64-bit integers, to both ends of their range
    for (int rep = 0; rep < 3000 && p < (1ull << 28); ++rep) {
        const int terms = rep % 3 == 0 ? kMacTermsLazy : kMacTerms;
        int64_t sum = rep % 7 == 0 ? (1ll << 28) - 1 : rep % 7 == 1 ? -(1ll << 28) + 1 : rnd_signed(29);
        i128 exact = sum;
        for (int i = 0; i < terms; ++i) {
            int64_t x = (int64_t)(rnd() % p), k = (int64_t)(rnd() % p);
            if (rep % 5 == 0) x = p - 1;
            if (rep % 3 == 0) k = rep % 5 == 0 ? (int64_t)(0.51 * p) * (rep & 1 ? -1 : 1) : k / 2 - (int64_t)(p / 4);
            else if (rep % 5 == 0) k = rep & 1 ? -(int64_t)p : (int64_t)p;
            mac_int((int32_t)x, (int32_t)k, sum);
            exact += (i128)x * k;
        }
        CHECK((i128)sum == exact, "mac_int sum of %d terms", terms);
        const double q = __builtin_rint((double)(int32_t)(sum >> 32) * 4294967296.0 * m.pinv);
        CHECK(fabs(q) <= 250.0 * (double)p && fabs(q) < 68719476736.0, "mac_int quotient");
        const double r = mac_int_reduce(sum, m);
        CHECK(fabs(r) <= lim && mod_i128((i128)(int64_t)r, p) == mod_i128(exact, p), "mac_int_reduce");
    }
    // split3: the pieces add up, have the stated granularity and magnitude; with the centred shifted factors, seventeen
    // sources accumulate exactly and reduce to sum y_i f_i mod p
    for (int rep = 0; rep < 20000; ++rep) {
        double acc = 0.0;
        i128 exact = 0;
        for (int i = 0; i < 17; ++i) {
            int64_t y = rnd() >> 28;  // below 2^36
            if (rep % 9 == 0) y = (uint64_t[]){0, (1ull << 36) - 1, (1ull << 24) - 1, 1ull << 23, (1ull << 23) + (1ull << 11), p - 1, 0xFFF800800ull, 0x800800ull}[(rep / 9 + i) % 8];
            if (i == 16) y = -(y / 2);  // the signed remainder of a rescale
            uint64_t f = rnd() % p;
            if (rep % 5 == 0) f = (i & 1) ? p / 2 : p / 2 + 1;  // largest centred magnitudes
            double y2, y1, y0;
            split3((double)y, y2, y1, y0);
            CHECK(y2 + y1 + y0 == (double)y, "split3 sum %llu", (unsigned long long)y);
            CHECK(fmod(y2, 16777216.0) == 0 && (y2 >= 0 || i == 16) && fabs(y2) <= 68719476736.0, "split3 y2 %llu", (unsigned long long)y);
            CHECK(fmod(y1, 4096.0) == 0 && fabs(y1) <= 8388608.0, "split3 y1 %llu", (unsigned long long)y);
            CHECK(fabs(y0) <= 2048.0 && y0 == floor(y0), "split3 y0 %llu", (unsigned long long)y);
            double fk[3];
            for (int k = 0; k < 3; ++k) {
                const uint64_t s = (uint64_t)(((i128)f << (12 * k)) % p);
                fk[k] = ldexp(s > p / 2 ? -(double)(p - s) : (double)s, -12 * k);
            }
            acc = __builtin_fma(y2, fk[2], __builtin_fma(y1, fk[1], __builtin_fma(y0, fk[0], acc)));
            CHECK(acc == floor(acc) && fabs(acc) < 9007199254740992.0, "split3 accumulator not an exact integer");
            exact += (i128)y * f;
        }
        const double r = reduce_lazy(acc, m);
        CHECK(fabs(r) <= lim && mod_i128((i128)(int64_t)r, p) == mod_i128(exact, p), "split3 conversion sum");
    }
    // split2 (contexts whose moduli are all below 2^32): the two pieces add up, have the stated granularity and magnitude;
    // with the centred factors cut at 16 bits, seventeen sources accumulate exactly and reduce to sum y_i f_i mod p
    if (p < (1ull << 32)) {
        for (int rep = 0; rep < 20000; ++rep) {
            double acc = 0.0;
            i128 exact = 0;
            for (int i = 0; i < 17; ++i) {
                int64_t y = rnd() >> 32;  // below 2^32: a residue of some other modulus of such a context
                if (rep % 9 == 0) y = (uint64_t[]){0, (1ull << 32) - 1, (1ull << 16) - 1, 1ull << 15, (1ull << 15) + 1, p - 1, 0xFFFF8000ull, 0x8000ull}[(rep / 9 + i) % 8];
                if (i == 16) y = -(y / 2);
                uint64_t f = rnd() % p;
                if (rep % 5 == 0) f = (i & 1) ? p / 2 : p / 2 + 1;  // largest centred magnitudes
                double y1, y0;
                split2((double)y, y1, y0);
                CHECK(y1 + y0 == (double)y, "split2 sum %llu", (unsigned long long)y);
                CHECK(fmod(y1, 65536.0) == 0 && (y1 >= 0 || i == 16) && fabs(y1) <= 4294967296.0, "split2 y1 %llu", (unsigned long long)y);
                CHECK(fabs(y0) <= 32768.0 && y0 == floor(y0), "split2 y0 %llu", (unsigned long long)y);
                double fk[2];
                for (int k = 0; k < 2; ++k) {
                    const uint64_t s = (uint64_t)(((i128)f << (16 * k)) % p);
                    fk[k] = ldexp(s > p / 2 ? -(double)(p - s) : (double)s, -16 * k);
                }
                acc = __builtin_fma(y1, fk[1], __builtin_fma(y0, fk[0], acc));
                CHECK(acc == floor(acc) && fabs(acc) < 9007199254740992.0, "split2 accumulator not an exact integer below 2^53");
                exact += (i128)y * f;
            }
            const double r = reduce_lazy(acc, m);
            CHECK(fabs(r) <= lim && mod_i128((i128)(int64_t)r, p) == mod_i128(exact, p), "split2 conversion sum");
        }
    }
    // sixteen-point passes against exact butterflies; growth bounds
    for (int rep = 0; rep < 2000; ++rep) {
        double t[16], v[16], w[16];
        int64_t e[16];
        t[0] = 0;
        for (int k = 1; k < 16; ++k) t[k] = (double)(rnd() % p);
        for (int k = 0; k < 16; ++k) { e[k] = (rep & 1) ? (int64_t)(rnd() % p) : rnd_signed(40); v[k] = (double)e[k]; }
        double in_max = 0; for (int k = 0; k < 16; ++k) in_max = fmax(in_max, fabs(v[k]));
        // exact forward: stage u pairs k, k + (8 >> u) inside groups of 16 >> u
        int64_t x[16]; for (int k = 0; k < 16; ++k) x[k] = mod_i128(e[k], p);
        for (int u = 0; u < 4; ++u) { int half = 8 >> u; for (int g = 0; g < (1 << u); ++g) { int64_t tw = (int64_t)t[(1 << u) + g]; for (int i = 0; i < half; ++i) { int k = g * 2 * half + i; int64_t y = mod_i128((i128)x[k + half] * tw, p); int64_t a = x[k]; x[k] = mod_i128((i128)a + y, p); x[k + half] = mod_i128((i128)a - y, p); } } }
        for (int k = 0; k < 16; ++k) w[k] = v[k];
        radix16_fwd(w, t, m);
        for (int k = 0; k < 16; ++k) {
            CHECK(mod_i128((i128)(int64_t)w[k], p) == x[k], "radix16_fwd value");
            CHECK(fabs(w[k]) <= in_max + 4 * lim, "radix16_fwd growth");
        }
        // shortened passes (last 4 - U0 stages only) against the same exact butterflies
        {
            int64_t y[16];
            double z[16];
            for (int k = 0; k < 16; ++k) { y[k] = mod_i128(e[k], p); z[k] = v[k]; }
            for (int u = 2; u < 4; ++u) { int half = 8 >> u; for (int g = 0; g < (1 << u); ++g) { int64_t tw = (int64_t)t[(1 << u) + g]; for (int i = 0; i < half; ++i) { int k = g * 2 * half + i; int64_t xx = mod_i128((i128)y[k + half] * tw, p); int64_t a = y[k]; y[k] = mod_i128((i128)a + xx, p); y[k + half] = mod_i128((i128)a - xx, p); } } }
            radix16_fwd<2>(z, t, m);
            for (int k = 0; k < 16; ++k) CHECK(mod_i128((i128)(int64_t)z[k], p) == y[k], "radix16_fwd<2> value");
            for (int k = 0; k < 16; ++k) { y[k] = mod_i128(e[k], p); z[k] = v[k]; }
            for (int u = 3; u >= 1; --u) { int half = 8 >> u; for (int g = 0; g < (1 << u); ++g) { int64_t tw = (int64_t)t[(1 << u) + g]; for (int i = 0; i < half; ++i) { int k = g * 2 * half + i; int64_t a = y[k], b = y[k + half]; y[k] = mod_i128((i128)a + b, p); y[k + half] = mod_i128((i128)mod_i128((i128)a - b, p) * tw, p); } } }
            if (rep & 1) {   // canonical inputs: inside the inverse pass's input range
                radix16_inv<1>(z, t, m);
                for (int k = 0; k < 16; ++k) CHECK(mod_i128((i128)(int64_t)z[k], p) == y[k], "radix16_inv<1> value");
            }
        }
        // inverse pass needs |v| <= p
        for (int k = 0; k < 16; ++k) { e[k] = (int64_t)(rnd() % (2 * p)) - (int64_t)p; v[k] = (double)e[k]; x[k] = mod_i128(e[k], p); }
        for (int u = 3; u >= 0; --u) { int half = 8 >> u; for (int g = 0; g < (1 << u); ++g) { int64_t tw = (int64_t)t[(1 << u) + g]; for (int i = 0; i < half; ++i) { int k = g * 2 * half + i; int64_t a = x[k], b = x[k + half]; x[k] = mod_i128((i128)a + b, p); x[k + half] = mod_i128((i128)(a - b) * tw, p); } } }
        radix16_inv(v, t, m);
        for (int k = 0; k < 16; ++k) {
            CHECK(mod_i128((i128)(int64_t)v[k], p) == x[k], "radix16_inv value");
            CHECK(fabs(v[k]) <= 16.0 * (double)p, "radix16_inv growth");
        }
    }
}

// Primes = 1 (mod 2^13) below 2^bits, largest first.
static std::vector<uint64_t> primes_below(int bits, int count) {
    std::vector<uint64_t> found;
    for (uint64_t p = (1ull << bits) - 8191; (int)found.size() < count; p -= 8192) {
        bool prime = true;
        for (uint64_t d = 3; prime && d * d <= p; d += 2) prime = p % d != 0;
        if (prime) found.push_back(p);
    }
    return found;
}

// The fused conversions as the kernels compute them, from the library's own tables: sources in the bytes that they have in memory, summed
// in doubles (cut_source) and as the digit planes of the matrix cores, against sum y_i f_i.
template <int PIECES>
static void check_conversion(int bits, uint32_t n_src, uint32_t n_extra) {
    const uint32_t n_dst = 9, n_basis = n_src - n_extra;
    ks_ctx c;
    c.mod = primes_below(bits, (int)(n_src + n_dst));
    c.pieces = PIECES;
    std::vector<uint32_t> src, dst;
    std::vector<uint16_t> src_limb, dst_limb;
    for (uint32_t i = 0; i < n_src; ++i) { src.push_back(i); src_limb.push_back((uint16_t)i); }
    for (uint32_t t = 0; t < n_dst; ++t) { dst.push_back(n_src + t); dst_limb.push_back((uint16_t)t); }
    std::vector<BConvPlan> plans(1);
    BConvPlan& plan = plans[0];
    fill_bconv_plan(&c, &plan, src.data(), src_limb.data(), n_src, dst.data(), dst_limb.data(), n_dst, 0, n_extra);
    // the largest sum that the cut admits: every piece and every factor at its end
    const double f = ldexp(1.0, bits - 1), most = PIECES == 3 ? 4095 * f + 16773120.0 * f / 4096 + (4096 + 128) * f : 65535 * f + (65536 + 32896) * f;
    CHECK(17 * most + f < 9007199254740992.0, "bound of the sums of %d pieces at %d bits", PIECES, bits);
    for (int rep = 0; rep < 2000; ++rep) {
        std::vector<int64_t> y(n_src);
        for (uint32_t i = 0; i < n_src; ++i) {
            const int64_t s = (int64_t)c.mod[i];
            y[i] = (int64_t)(rnd() % (uint64_t)s);
            if (rep % 4 == 0) y[i] = (int64_t[]){0, s - 1, 0x7F7F7F80, 0x7F7F7F7F, 0xFFFFFF, (s >> 24 << 24) - 0x80808081ll, 1, s / 2}[(rep / 4 + i) % 8];
            if (y[i] < 0 || y[i] >= s) y[i] = s - 1;
            if (i >= n_basis) y[i] = rep % 4 == 1 ? -(s / 2) : rep % 4 == 2 ? s / 2 : y[i] - s / 2;   // signed
        }
        std::vector<uint32_t> word(n_src);
        std::vector<int> top(n_src);
        for (uint32_t i = 0; i < n_src; ++i) {
            const double biased = (double)y[i] + kDigitBias;
            uint64_t raw;
            memcpy(&raw, &biased, 8);
            word[i] = (uint32_t)raw;
            top[i] = (int)(int8_t)(raw >> 32);
        }
        for (uint32_t t = 0; t < n_dst; ++t) {
            const Mod m = plan.dst_mod[t];
            const int64_t mt = (int64_t)c.mod[dst[t]];
            i128 exact = 0;
            double acc = plan.dst_start[t];
            for (uint32_t i = 0; i < n_src; ++i) {
                int64_t prod = 1;
                for (uint32_t k = 0; k < n_basis; ++k)
                    if (k != i) prod = mod_i128((i128)prod * (int64_t)c.mod[k], mt);
                exact += (i128)y[i] * prod;
                double piece[PIECES];
                cut_source<PIECES>(word[i], top[i], piece);
                for (int k = 0; k < PIECES; ++k) {
                    acc = __builtin_fma(piece[k], plan.hats[t][i][k + 1 < PIECES ? k : 3], acc);
                    CHECK(acc == floor(acc) && fabs(acc) < 9007199254740992.0, "conversion sum, %d pieces", PIECES);
                }
            }
            const int64_t want = mod_i128(exact, mt);
            CHECK(mod_i128((i128)(int64_t)reduce_lazy(acc, m), mt) == want, "conversion, %d pieces of %u sources at %d bits", PIECES, n_src, bits);
            int64_t planes[kMfmaPlanes] = {};
            for (int slot = 0; slot < 2 * mfma_instructions((int)plan.mfma_t); ++slot)
                for (int e = 0; e < mfma_slot_sources((int)plan.mfma_t, slot / 2); ++e) {
                    const uint32_t i = plan.mfma_src_limb[3 * slot + e];
                    for (int b = 0; b < kMfmaPlanes; ++b) {
                        const int8_t* row = plan.afac[t][b][slot];
                        for (int a = 0; a < 4; ++a) planes[b] += row[4 * e + a] * (int)(int8_t)((word[i] >> (8 * a) & 255u) ^ 128u);
                        planes[b] += row[12 + e] * top[i];
                    }
                }
            int64_t v = 0;
            for (int b = kMfmaPlanes - 1; b >= 0; --b) {
                CHECK(llabs(planes[b]) <= 17ll * 5 * (1 << 14), "digit plane %d", b);
                v = v * 256 + planes[b];
            }
            CHECK(llabs(planes[0] + planes[1] * 256) < (1ll << 31) && llabs(planes[2] + planes[3] * 256) < (1ll << 31), "pairs of digit planes");
            CHECK(llabs(v) < (1ll << 49) && mod_i128((i128)(int64_t)reduce_lazy((double)v, m), mt) == want, "digit planes of %u sources at %d bits", n_src, bits);
        }
    }
}

// The units of the rotation gathers go to eight XCDs in rounds: the last round leaves at most an eighth of all places idle.
static void check_gather_parts() {
    for (uint32_t E = 4; E <= 255; ++E) {
        const uint32_t units = E << gather_parts_log(E), places = (units + 7) / 8 * 8;
        CHECK((places - units) * 8 <= places, "%u limb positions: %u of %u places idle", E, places - units, places);
    }
}

// The targets per workgroup of a conversion follow from the workgroups that have work: digits of different sizes and of one size alike
// that hold the same number of targets.
static void check_conversion_targets() {
    const uint32_t lines[] = {1024, 8192};
    const int below[] = {1, 2}, above[] = {2, 4};
    for (int i = 0; i < 2; ++i)
        for (uint32_t tiles = 1; tiles <= 16; tiles *= 2)
            for (uint32_t plans = 1; plans <= 4; ++plans)
                for (uint32_t most = 1; most <= 40; ++most)
                    for (uint32_t last = plans == 1 ? most : 1; last <= most; ++last) {
                        PlanSet set;
                        set.n_plans = plans;
                        set.max_targets = most;
                        set.targets = (plans - 1) * most + last;
                        const uint32_t per_poly = tiles * set.targets, polys = lines[i] / per_poly;
                        if (polys == 0 || per_poly > lines[i]) continue;
                        CHECK(vector_conversion_targets(set, tiles, polys) == below[i], "%u plans of %u and %u targets, %u tiles, %u polynomials", plans, most, last, tiles, polys);
                        CHECK(vector_conversion_targets(set, tiles, polys + 1) == above[i], "%u plans of %u and %u targets, %u tiles, %u polynomials", plans, most, last, tiles, polys + 1);
                    }
}

int main() {
    check_gather_parts();
    check_conversion_targets();
    for (uint32_t n_src : {1u, 2u, 5u, 8u, 13u, 16u, 17u}) {
        const uint32_t n_extra = n_src == 17 || n_src == 2 ? 1 : 0;
        check_conversion<3>(36, n_src, n_extra);
        check_conversion<2>(32, n_src, n_extra);
        check_conversion<2>(28, n_src, n_extra);
    }
    const uint64_t primes[] = {68718428161ull /* largest, N=2^16 */, 68617633793ull /* 60th, N=2^16 */, 68719403009ull /* largest, N=2^12 */,
                               68718764033ull /* 6th, N=2^12 */, 34359754753ull /* a 35-bit prime = 1 mod 2^17 */,
                               // the rest of the admitted range: the paper's word size, the top of the 32-bit range, a tiny modulus
                               268042241ull /* largest 28-bit prime = 1 mod 2^17 */, 4293918721ull /* largest below 2^32, = 1 mod 2^17 */,
                               40961ull /* = 1 mod 2^13 */};
    for (uint64_t p : primes) check_prime(p);
    if (fails) { printf("%d checks failed\n", fails); return 1; }
    printf("OK\n");
    return 0;
}
