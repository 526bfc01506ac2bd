// Slot-wise kernels (Kernel Code Generation, "Elementwise" kernel class): inner products with evaluation keys through the
// evaluation-domain automorphism (gathers).  One thread per slot, contiguous segments per wavefront,
// operands shared by both key components and by all ciphertexts of a group are read once ("load reuse").
#include "ks_gather.hpp"

namespace ks {

// What one sum of the gather kernels takes at most: the digits of a rotation, and with lazy factors those of all rotations of a
// launch and their c0.
static_assert(kMaxDigits <= kMacTerms && kMacRotations * (kMaxDigits + 1) <= kMacTermsLazy, "products per exact sum");

// Inner products through the sigma_g gather for a group of hoisted rotations: acc[r][b][c][pos] = sum_j sigma_{g_r}(src_j)[pos]
// key_r[j][c][pos].  One thread owns one slot of one limb position for all ciphertexts of the group and walks the
// rotations of the launch; the operands of the next (rotation, digit) are requested before the current products.
// WK: word type of the keys; PACKED: the bundle's sources have bits above 32.
// Four rotations of 8 ciphertexts, N = 2^16, E = 32, three digits: 350 -> 320 us, 1.4 GB of compulsory traffic.
// The result is packed ([r][b][2][E] limbs in rows order).
// pos0: first limb position of the launch (0, or ell where the others' sums meet the division).
template <int G, typename WK, bool PACKED, bool INT>
__global__ __launch_bounds__(256, 4) void inner_product_kernel(const Mod* __restrict__ mods, uint32_t ell, uint32_t E, uint32_t L, uint32_t M,
                                                            uint32_t logN, uint32_t ndig, uint32_t pos0, uint32_t parts_log, GatherBundle src,
                                                            MacRotations rot, uint8_t* __restrict__ acc) {
    using Sum = MacSum<INT>;
    using Factor = typename Sum::Factor;
    const uint32_t N = 1u << logN;
    const GatherTile tile = gather_tile(E - pos0, logN, parts_log, threadIdx.x);
    if (!tile.valid) return;  // uniform
    const uint32_t pos = pos0 + tile.pos, n = tile.n, mid = pos < ell ? pos : L + (pos - ell);
    const Mod m = mods[mid];
    const BundleRsrc bundle = bundle_rsrc<G>(src, (uint64_t)ndig * E * N);
    struct Raw {
        SlotRaw<G> x;
        WK k0, k1;
    };
    auto fetch = [&](uint32_t r, uint32_t j) {
        Raw w;
        const uint32_t sn = galois_source_slot(n, rot.galois[r], logN);
        // a key is below 4 GB: [8][2][255][2^16] words of at most 8 bytes
        const BufferRsrc key = uniform_rsrc(rot.key[r], (uint64_t)ndig * 2 * M * N * sizeof(WK));
        const uint32_t at = (j * 2 * M + mid) * N * (uint32_t)sizeof(WK);
        w.k0 = buffer_load<WK>(key, n * (uint32_t)sizeof(WK), at);
        w.k1 = buffer_load<WK>(key, n * (uint32_t)sizeof(WK), at + M * N * (uint32_t)sizeof(WK));
        w.x = slot_load<G, PACKED>(bundle, j * E + pos, N, sn);
        return w;
    };
    Raw cur = fetch(0, 0);
    const uint32_t element = packed_element(n & ~63u);
#pragma unroll 1
    for (uint32_t r = 0; r < rot.n; ++r) {
        Sum s0[G], s1[G];
#pragma unroll
        for (int b = 0; b < G; ++b) {
            s0[b].start(0.0);
            s1[b].start(0.0);
        }
#pragma unroll 1
        for (uint32_t j = 0; j < ndig; ++j) {
            const bool last = j + 1 == ndig;
            const Raw next = fetch(last ? min(r + 1, rot.n - 1) : r, last ? 0 : j + 1);
            const Factor k0 = Sum::template word<WK>(cur.k0), k1 = Sum::template word<WK>(cur.k1);
            const SlotRaw<G> s = slot_take<G, PACKED>(cur.x);
#pragma unroll
            for (int b = 0; b < G; ++b) {
                const Factor x = Sum::template source<G, PACKED>(s, b);
                s0[b].add(x, k0);
                s1[b].add(x, k1);
                // the second half's sources become doubles after the first half's products: all eight at once spilled two registers
                // (32-bit moduli, eight rotations of eight ciphertexts, N = 2^16: 2278 -> 2265 us; N = 2^12 65.2 -> 64.1)
                if (!PACKED && !INT && b == 3) __builtin_amdgcn_sched_barrier(0);
            }
            cur = next;
        }
        uint8_t* ar = acc + ((uint64_t)r * G * 2 * E + pos) * packed_limb_bytes(N);
        double sums[2 * G];
#pragma unroll
        for (int b = 0; b < G; ++b) {
            sums[2 * b] = s0[b].reduce(m);
            sums[2 * b + 1] = s1[b].reduce(m);
        }
        packed_put<2 * G>(ar, E * packed_limb_bytes(N), N, element, sums);
    }
}

// LAUNCH(group, word type of the keys, PACKED, INT)
#define KS_GATHER_INT(GV) KS_GATHER_LAUNCH(GV, uint32_t, false, true)
#define KS_GATHER_32(GV) KS_GATHER_LAUNCH(GV, uint32_t, false, false)
#define KS_GATHER_PACKED_32(GV) KS_GATHER_LAUNCH(GV, uint32_t, true, false)
#define KS_GATHER_PACKED_64(GV) KS_GATHER_LAUNCH(GV, uint64_t, true, false)
#define KS_FOR_GATHER_KERNEL()                                             \
    if (!src.hi && integer_sums(c)) { KS_FOR_GROUP(src.group, KS_GATHER_INT) } \
    else if (!src.hi) { KS_FOR_GROUP(src.group, KS_GATHER_32) }            \
    else if (key_words32) { KS_FOR_GROUP(src.group, KS_GATHER_PACKED_32) } \
    else { KS_FOR_GROUP(src.group, KS_GATHER_PACKED_64) }

void launch_inner_product(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, uint8_t* acc,
                          hipStream_t s, bool key_words32, bool special_only) {
    if (rot.n == 0) return;
    const uint32_t batch = src.group;
    const uint32_t pos0 = special_only ? lv.ell : 0, n_pos = lv.E - pos0, pl = gather_parts_log(n_pos);
    // reads: every raised digit limb per ciphertext once per launch, each rotation's key once; writes: both accumulators of
    // every rotation
    const double wk = key_words32 ? 4.0 : 8.0;
    ProfScope ps("inner_product",
                 (src_bytes(src) * batch * lv.ndig + (double)rot.n * (wk * 2.0 * lv.ndig + 10.0 * batch)) * n_pos * c->N,
                 s);
#define KS_GATHER_LAUNCH(GV, WKT, PK, IS)                                                                                                     \
    hipLaunchKernelGGL((inner_product_kernel<GV, WKT, PK, IS>), dim3(gather_grid(c, n_pos, pl)), dim3(256), 0, s, c->d_mod, lv.ell, lv.E, c->L, \
                       c->M, c->logN, lv.ndig, pos0, pl, src, rot, acc)
    KS_FOR_GATHER_KERNEL()
#undef KS_GATHER_LAUNCH
}

// Rotate-multiply-accumulate on the extended basis (inner sum of a baby-step giant-step transform with the division by P
// deferred to the whole sum).  One thread owns one slot of one limb position for all ciphertexts of the group; the two
// running sums of each stay in registers as exact integers (mac_exact) until every rotation of the launch is in.  The digits
// are the OUTER loop and the rotations the inner one, so that between two rotations only one digit's slots are gathered from
// and about half of them are found in the XCD's L2 (see gather_tile); each key slot and each plaintext slot is still read once (the
// plaintext slots stay in LDS).  The operands of the next (digit, rotation) are requested before the current products.
// 8 ciphertexts x 16 keyed rotations, three digits, N = 2^16, E = 32: 656 us (28-bit moduli, integer sums, 417), where one thread per slot that
// walked digits inside rotations and gathered each ciphertext on its own took 1037 (9.6 GB through the fabric, now 3.3).
// What bounds it: the stream of keys and plaintexts (1.9 of 3.1 GB read) and fp64 issue (61 % of the slots), partly overlapped.
// Three wavefronts per SIMD (integer sums four): squeezed into 128 registers for a fourth, the few spilled words cost more fabric traffic than
// the occupancy gains (40-100 us more).  Sixteen ciphertexts per launch sharing the key reads measured the same per ciphertext:
// what the shared keys save, the doubled sources lose in L2.
// rot: the n_key rotations that take a key come first, then the identities (the term P (c0, c1), no key read).
template <int G, typename WK, bool PACKED, bool INT>
__global__ __launch_bounds__(256, INT ? 4 : 3) void rotate_mac_kernel(const Mod* __restrict__ mods, const double* __restrict__ Pmod, uint32_t ell,
                                                         uint32_t E, uint32_t L, uint32_t M, uint32_t logN, DigitRanges dg,
                                                         uint32_t parts_log, GatherBundle src, MacRotations rot, uint32_t n_key,
                                                         uint8_t* __restrict__ u, int accumulate) {
    using Sum = MacSum<INT>;
    using Factor = typename Sum::Factor;
    const uint32_t N = 1u << logN;
    const GatherTile tile = gather_tile(E, logN, parts_log, threadIdx.x);
    if (!tile.valid) return;  // uniform
    const uint32_t pos = tile.pos, n = tile.n, mid = pos < ell ? pos : L + (pos - ell);
    const Mod m = mods[mid];
    const BundleRsrc bundle = bundle_rsrc<G>(src, ((uint64_t)dg.ndig * E + ell) * N);
    const uint32_t element = packed_element(n);
    uint8_t* up = u + (uint64_t)pos * packed_limb_bytes(N);
    const uint64_t comp = E * packed_limb_bytes(N);
    Sum s0[G], s1[G];
#pragma unroll
    for (int b = 0; b < G; ++b) {
        s0[b].start(accumulate ? packed_get(up + 2 * b * comp, N, element) : 0.0);
        s1[b].start(accumulate ? packed_get(up + (2 * b + 1) * comp, N, element) : 0.0);
    }
    struct Raw {
        SlotRaw<G> x;
        WK k0, k1;
    };
    auto fetch = [&](uint32_t j, uint32_t r) {
        Raw w;
        const uint32_t sn = galois_source_slot(n, rot.galois[r], logN);
        // a key is below 4 GB: [8][2][255][2^16] words of at most 8 bytes
        const BufferRsrc key = uniform_rsrc(rot.key[r], (uint64_t)dg.ndig * 2 * M * N * sizeof(WK));
        const uint32_t at = (j * 2 * M + mid) * N * (uint32_t)sizeof(WK);
        w.x = slot_load<G, PACKED>(bundle, j * E + pos, N, sn);
        w.k0 = buffer_load<WK, 2>(key, n * (uint32_t)sizeof(WK), at);
        w.k1 = buffer_load<WK, 2>(key, n * (uint32_t)sizeof(WK), at + M * N * (uint32_t)sizeof(WK));
        return w;
    };
    Raw qa;
    if (n_key != 0) qa = fetch(0, 0);
    // The plaintext slots are used once per digit and once more for c0: each thread keeps its own in LDS (a null plaintext is the
    // constant 1).  Read from memory every time they were 0.8 of 3.3 GB of a launch.
    extern __shared__ uint64_t pts_lds[];
    auto pts = [&](uint32_t r) { return reinterpret_cast<WK*>(pts_lds) + r * 256 + threadIdx.x; };
#pragma unroll 1
    for (uint32_t r0 = 0; r0 < rot.n; r0 += 8) {
        WK w[8];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) {
            const void* pt = r0 + i < rot.n ? rot.pt[r0 + i] : nullptr;   // (places past the last rotation are read against a factor of zero)
            w[i] = pt ? buffer_load<WK>(uniform_rsrc(pt, (uint64_t)M * N * sizeof(WK)), n * (uint32_t)sizeof(WK), mid * N * (uint32_t)sizeof(WK)) : (WK)1;
        }
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) *pts(r0 + i) = w[i];
    }
    if (n_key != 0) {
        const uint32_t steps = dg.ndig * n_key;
        uint32_t j = 0, r = 0;
        auto advance = [&]() {  // to the next (digit, rotation); stays on the last one at the end
            if (r + 1 < n_key) ++r;
            else if (j + 1 < dg.ndig) { r = 0; ++j; }
        };
        auto products = [&](const Raw& q, uint32_t rq) {
            // the plaintext slot is folded into the key slots, not multiplied per ciphertext
            const double w = word_to_f64<WK>(*pts(rq));
            const Factor k0 = Sum::factor(mulmod_lazy(word_to_f64<WK>(q.k0), w, m)), k1 = Sum::factor(mulmod_lazy(word_to_f64<WK>(q.k1), w, m));
            const SlotRaw<G> s = slot_take<G, PACKED>(q.x);
#pragma unroll
            for (int b = 0; b < G; ++b) {
                const Factor x = Sum::template source<G, PACKED>(s, b);
                s0[b].add(x, k0);
                s1[b].add(x, k1);
            }
        };
        // two steps a trip: operands and sums alternate between two register sets instead of being copied
#pragma unroll 1
        for (uint32_t t = 0; t + 1 < steps; t += 2) {
            const uint32_t ra = r;
            advance();
            const uint32_t rb = r;
            const Raw qb = fetch(j, r);
            products(qa, ra);
            advance();
            qa = fetch(j, r);
            products(qb, rb);
        }
        if (steps & 1) products(qa, r);  // (a break inside the loop costs it 2-5 %)
    }
    if (pos < ell) {  // uniform: P c0 of every rotation, P c1 of the identities
        const double pm = Pmod[pos];
        uint32_t own = 0;
        while (own + 1 < dg.ndig && pos >= dg.hi[own]) ++own;
        if (src.c0) {  // uniform
            using WC = std::conditional_t<PACKED, uint64_t, uint32_t>;
#pragma unroll 1
            for (uint32_t r = 0; r < rot.n; ++r) {
                const WC* cp = static_cast<const WC*>(src.c0) + (uint64_t)pos * N + (r < n_key ? galois_source_slot(n, rot.galois[r], logN) : n);
                WC x[G];
#pragma unroll
                for (int b = 0; b < G; ++b) x[b] = cp[b * src.c0_ps];
                const Factor pw = Sum::factor(mulmod_lazy(pm, word_to_f64<WK>(*pts(r)), m));
#pragma unroll
                for (int b = 0; b < G; ++b) s0[b].add(Sum::template word<WC>(x[b]), pw);
            }
        } else {
            constexpr uint32_t AHEAD = 2;  // rotations in flight
            SlotRaw<G> x[AHEAD];
            auto fetch0 = [&](uint32_t r, int i) {
                r = min(r, rot.n - 1);
                x[i] = slot_load<G, PACKED>(bundle, dg.ndig * E + pos, N, r < n_key ? galois_source_slot(n, rot.galois[r], logN) : n);
            };
#pragma unroll
            for (uint32_t i = 0; i < AHEAD; ++i) fetch0(i, i);
#pragma unroll 1
            for (uint32_t r0 = 0; r0 < rot.n; r0 += AHEAD) {
#pragma unroll
                for (uint32_t i = 0; i < AHEAD; ++i) {
                    const Factor pw = Sum::factor(mulmod_lazy(r0 + i < rot.n ? pm : 0.0, word_to_f64<WK>(*pts(r0 + i)), m));
                    const SlotRaw<G> s = slot_take<G, PACKED>(x[i]);
#pragma unroll
                    for (int b = 0; b < G; ++b) s0[b].add(Sum::template source<G, PACKED>(s, b), pw);
                    fetch0(r0 + i + AHEAD, i);
                }
            }
        }
#pragma unroll 1
        for (uint32_t r = n_key; r < rot.n; ++r) {
            const SlotRaw<G> x = slot_load<G, PACKED>(bundle, own * E + pos, N, n);
            const Factor pw = Sum::factor(mulmod_lazy(pm, word_to_f64<WK>(*pts(r)), m));
#pragma unroll
            for (int b = 0; b < G; ++b) s1[b].add(Sum::template source<G, PACKED>(x, b), pw);
        }
    }
    double sums[2 * G];
#pragma unroll
    for (int b = 0; b < G; ++b) {
        sums[2 * b] = s0[b].reduce(m);
        sums[2 * b + 1] = s1[b].reduce(m);
    }
    packed_put<2 * G>(up, comp, N, packed_element(n & ~63u), sums);
}

void launch_rotate_mac(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, uint8_t* u,
                       bool accumulate, hipStream_t s, bool key_words32) {
    if (rot.n == 0) return;
    const uint32_t batch = src.group;
    const uint32_t pl = gather_parts_log(lv.E);
    DigitRanges dg;
    dg.ndig = lv.ndig;
    for (uint32_t j = 0; j < kMaxDigits; ++j) {
        dg.lo[j] = j < lv.ndig ? lv.digit_lo[j] : 0;
        dg.hi[j] = j < lv.ndig ? lv.digit_hi[j] : 0;
    }
    MacRotations sorted = rot;
    uint32_t n_key = 0, n_id = 0;
    for (int pass = 0; pass < 2; ++pass)
        for (uint32_t r = 0; r < rot.n; ++r) {
            if ((rot.galois[r] == 1) != (pass == 1)) continue;
            const uint32_t to = n_key + n_id;
            sorted.galois[to] = rot.galois[r];
            sorted.key[to] = rot.key[r];
            sorted.pt[to] = rot.pt[r];
            ++(pass == 0 ? n_key : n_id);
        }
    // Algorithmic traffic: the raised digits and c0 of a ciphertext once (the rotations of a launch re-read them through
    // the gather; those re-reads are meant to come from cache), key and plaintext of every rotation once, both sums written
    // once.  Algorithmic work per slot, ciphertext and rotation: 2 NDIG + 1 exact products (+ 2 NDIG + 1 modular ones per group).
    const double reads = batch * src_bytes(src) * (lv.ndig * lv.E + lv.ell) + (key_words32 ? 4.0 : 8.0) * (double)rot.n * (2.0 * lv.ndig + 1.0) * lv.E;
    ProfScope ps("rotate_mac", (reads + (double)batch * 10 * lv.E * (accumulate ? 2 : 1)) * c->N, s,
                 (double)rot.n * lv.E * c->N * (4.0 * batch + 6.0) * (2 * lv.ndig + 1));
    // LDS for the plaintext slots, in rows of eight rotations: 16 KB a workgroup for five rotations in 64-bit words leave the small groups
    // the occupancy that a fixed 32 KB took from them (one ciphertext, 17 limbs, 28 bits: 76 -> 55 us; 36 bits 105 -> 92)
    const uint32_t lds_words = (rot.n + 7) / 8 * 8 * 256;
#define KS_GATHER_LAUNCH(GV, WKT, PK, IS)                                                                                                     \
    hipLaunchKernelGGL((rotate_mac_kernel<GV, WKT, PK, IS>), dim3(gather_grid(c, lv.E, pl)), dim3(256), lds_words * sizeof(WKT), s, c->d_mod, c->d_Pmod, lv.ell, lv.E, \
                       c->L, c->M, c->logN, dg, pl, src, sorted, n_key, u, accumulate ? 1 : 0)
    KS_FOR_GATHER_KERNEL()
#undef KS_GATHER_LAUNCH
#undef KS_FOR_GATHER_KERNEL
#undef KS_GATHER_32
#undef KS_GATHER_INT
#undef KS_GATHER_PACKED_32
#undef KS_GATHER_PACKED_64
}

}  // namespace ks
