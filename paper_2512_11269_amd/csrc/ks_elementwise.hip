// Slot-wise kernels (Kernel Code Generation, "Elementwise" kernel class): inner products with evaluation keys through the
// evaluation-domain automorphism (gathers).  One thread per slot, contiguous segments per wavefront,
// operands shared by both key components and by all ciphertexts of a group are read once ("load reuse").
#include <algorithm>

#include "ks_internal.hpp"
#include "ks_tiles.hpp"

namespace ks {

// What one sum of the gather kernels takes at most: the digits of a rotation, and with lazy factors those of all rotations of a
// launch and their c0.
static_assert(kMaxDigits <= kMacTerms && kMacRotations * (kMaxDigits + 1) <= kMacTermsLazy, "products per exact sum");

// One slot of a bundle slab as a gather loads it: the low words of the group's ciphertexts and the word of their bits above.
template <int G>
struct SlotRaw {
    uint32_t lo[G];
    uint32_t hi, from;
};
// Loads of the gather kernels go through buffer descriptors: a uniform byte offset in a scalar register plus one 32-bit
// byte offset per lane.  As 64-bit addresses per stream they pushed the sums out of the register file.
template <typename T, int CPOL = 0>
__device__ __forceinline__ T buffer_load(BufferRsrc rsrc, uint32_t lane_bytes, uint32_t uniform_bytes) {
    if constexpr (sizeof(T) == 16) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)lane_bytes, (int)uniform_bytes, CPOL));
    else if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)lane_bytes, (int)uniform_bytes, CPOL));
    else if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)lane_bytes, (int)uniform_bytes, CPOL));
    else if constexpr (sizeof(T) == 2) return (T)__builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)lane_bytes, (int)uniform_bytes, CPOL);
    else return (T)__builtin_amdgcn_raw_buffer_load_b8(rsrc, (int)lane_bytes, (int)uniform_bytes, CPOL);
}
// W consecutive 32-bit words
template <int W>
__device__ __forceinline__ void buffer_load_words(uint32_t* w, BufferRsrc rsrc, uint32_t lane_bytes, uint32_t uniform_bytes) {
    if constexpr (W == 3) {
        const auto t = __builtin_amdgcn_raw_buffer_load_b96(rsrc, (int)lane_bytes, (int)uniform_bytes, 0);
        w[0] = t[0]; w[1] = t[1]; w[2] = t[2];
    } else {
        struct alignas(4 * W) Words {
            uint32_t w[W];
        };
        const Words t = buffer_load<Words>(rsrc, lane_bytes, uniform_bytes);
#pragma unroll
        for (int k = 0; k < W; ++k) w[k] = t.w[k];
    }
}
// Descriptor of a tensor whose address is uniform, kept in scalar registers.
__device__ __forceinline__ BufferRsrc uniform_rsrc(const void* p, uint64_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32));
    const uint64_t u = (uint64_t)hi << 32 | lo;
    return make_buffer_rsrc(reinterpret_cast<const void*>(u), bytes);
}
// The bundle (below 4 GB: at most 192 + 192 slabs of 2^16 slots of 32 bytes).
struct BundleRsrc {
    BufferRsrc lo, hi;
};
template <int G>
__device__ __forceinline__ BundleRsrc bundle_rsrc(const GatherBundle& src, uint64_t slots) {
    return BundleRsrc{uniform_rsrc(src.lo, slots * (4 * G)), uniform_rsrc(src.hi, slots * gather_hi_bytes(G))};
}
// The slots sigma_g sends to a wavefront's 64 consecutive slots are one aligned block of 64, permuted.  The block is read
// in its own order and the lanes exchange what they hold on use (slot_take; 5 % on both kernels over permuted loads).
// slab: uniform; slot: the lane's source slot.
template <int G, bool PACKED>
__device__ __forceinline__ SlotRaw<G> slot_load(const BundleRsrc& src, uint32_t slab, uint32_t N, uint32_t slot) {
    using Layout = SlotLayout<G>;
    using HW = typename Layout::HW;
    const uint32_t block = slab * N + (__builtin_amdgcn_readfirstlane(slot) & ~63u), lane = threadIdx.x & 63u;
    SlotRaw<G> r;
    r.from = (slot & 63u) * 4;
    buffer_load_words<Layout::FIRST>(r.lo, src.lo, lane * (4 * Layout::FIRST), block * (4 * G));
    if constexpr (Layout::REST > 0) buffer_load_words<Layout::REST>(r.lo + 4, src.lo, lane * (4 * Layout::REST), block * (4 * G) + 1024);
    r.hi = PACKED ? buffer_load<HW>(src.hi, lane * (uint32_t)sizeof(HW), block * (uint32_t)sizeof(HW)) : 0u;
    return r;
}
__device__ __forceinline__ uint32_t from_lane(uint32_t v, uint32_t lane_bytes) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)lane_bytes, (int)v);
}
// the slot of this lane out of what the wavefront loaded
template <int G, bool PACKED>
__device__ __forceinline__ SlotRaw<G> slot_take(const SlotRaw<G>& l) {
    SlotRaw<G> r;
    r.from = l.from;
#pragma unroll
    for (int g = 0; g < G; ++g) r.lo[g] = from_lane(l.lo[g], l.from);
    r.hi = PACKED ? from_lane(l.hi, l.from) : 0u;
    return r;
}
template <int G, bool PACKED>
__device__ __forceinline__ double slot_f64(const SlotRaw<G>& r, int g) {
    return PACKED ? u64_to_f64((uint64_t)((r.hi >> (4 * g)) & 15u) << 32 | r.lo[g]) : (double)r.lo[g];
}

// The running sum of a gather kernel: exact products in two doubles, or in 64-bit integers (INT: unpacked slots, moduli below
// 2^28), where the slots are used as they come and a product is one instruction instead of four.
template <bool INT>
struct MacSum {
    double hi, lo;
    using Factor = double;
    __device__ __forceinline__ void start(double v) { hi = kMacBias; lo = v; }
    template <int G, bool PACKED>
    static __device__ __forceinline__ double source(const SlotRaw<G>& r, int g) { return slot_f64<G, PACKED>(r, g); }
    template <typename W>
    static __device__ __forceinline__ double word(W w) { return word_to_f64<W>(w); }
    static __device__ __forceinline__ double factor(double k) { return k; }
    __device__ __forceinline__ void add(double x, double k) { mac_exact(x, k, hi, lo); }
    __device__ __forceinline__ double reduce(Mod m) const { return mac_reduce(hi, lo, m); }
};
template <>
struct MacSum<true> {
    int64_t sum;
    using Factor = int32_t;
    __device__ __forceinline__ void start(double v) { sum = (int32_t)v; }
    template <int G, bool PACKED>
    static __device__ __forceinline__ int32_t source(const SlotRaw<G>& r, int g) { return (int32_t)r.lo[g]; }
    template <typename W>
    static __device__ __forceinline__ int32_t word(W w) { return (int32_t)w; }
    static __device__ __forceinline__ int32_t factor(double k) { return (int32_t)k; }
    __device__ __forceinline__ void add(int32_t x, int32_t k) { mac_int(x, k, sum); }
    __device__ __forceinline__ double reduce(Mod m) const { return mac_int_reduce(sum, m); }
};

// Workgroup -> (limb position, 256 slots) for the gather kernels.  Multiplication by a Galois element permutes the slots
// inside each half of a limb (g = 1 mod 4, every power of 5) or swaps the halves, so the sources of all rotations of a
// (position, half) are the bundle's slots of that position and half: 1.2 MB per digit for eight ciphertexts at N = 2^16,
// where the whole limb position of a chunk is 7 MB.  Consecutive workgroup ids go to the eight XCDs in turn, each with a
// 4 MB L2 of its own, so unit u = (position, part) goes to the workgroups of XCD u % 8, which walk one unit after the other:
// every rotation but the first finds its sources in that L2.  parts_log: gather_parts_log.
struct GatherTile {
    uint32_t pos, n;
    bool valid;
};
__device__ __forceinline__ GatherTile gather_tile(uint32_t E, uint32_t logN, uint32_t parts_log) {
    const uint32_t per_unit = 1u << (logN - 8 - parts_log), local = blockIdx.x >> 3;
    const uint32_t unit = (local / per_unit) * 8 + (blockIdx.x & 7);
    GatherTile t;
    t.valid = unit < (E << parts_log);
    t.pos = unit >> parts_log;
    t.n = (((unit & ((1u << parts_log) - 1)) * per_unit + local % per_unit) << 8) + (threadIdx.x & 255u);
    return t;
}
static uint32_t gather_grid(const ks_ctx* c, uint32_t E, uint32_t parts_log) {
    return (((E << parts_log) + 7) / 8) * 8 * ((c->N / 256) >> parts_log);
}

// Inner products through the sigma_g gather for a group of hoisted rotations: acc[r][b][c][pos] = sum_j sigma_{g_r}(src_j)[pos]
// key_r[j][c][pos].  One thread owns one slot of one limb position for all ciphertexts of the group and walks the
// rotations of the launch; the operands of the next (rotation, digit) are requested before the current products.
// WK: word type of the keys; PACKED: the bundle's sources have bits above 32.
// Four rotations of 8 ciphertexts, N = 2^16, E = 32, three digits: 350 -> 320 us, 1.4 GB of compulsory traffic.
// The result is packed ([r][b][2][E] limbs in rows order).
template <int G, typename WK, bool PACKED, bool INT>
__global__ __launch_bounds__(256, 4) void inner_product_kernel(const Mod* __restrict__ mods, uint32_t ell, uint32_t E, uint32_t L, uint32_t M,
                                                            uint32_t logN, uint32_t ndig, uint32_t parts_log, GatherBundle src,
                                                            MacRotations rot, uint8_t* __restrict__ acc) {
    using Sum = MacSum<INT>;
    using Factor = typename Sum::Factor;
    const uint32_t N = 1u << logN;
    const GatherTile tile = gather_tile(E, logN, parts_log);
    if (!tile.valid) return;  // uniform
    const uint32_t pos = tile.pos, n = tile.n, mid = pos < ell ? pos : L + (pos - ell);
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

// Integer sums: every modulus below 2^28 (250 products of a residue and a lazy one, 0.51 * 2^56 each, stay below 2^63).
// Eight ciphertexts, N = 2^16, E = 32, three digits, fp64 -> integer sums: calls of 16 rotations multiplied and summed 960 -> 869 us
// (82 registers instead of 134); at 28 bits no size was slower.
static bool integer_sums(const ks_ctx* c) {
    for (uint64_t m : c->mod)
        if (m >> 28) return false;
    return true;
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

// bytes a gathered source residue takes
static double src_bytes(const GatherBundle& g) { return g.hi ? 4.0 + (double)gather_hi_bytes(g.group) / g.group : 4.0; }

void launch_inner_product(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, uint8_t* acc,
                          hipStream_t s, bool key_words32) {
    if (rot.n == 0) return;
    const uint32_t batch = src.group;
    const uint32_t pl = gather_parts_log(lv.E);
    // reads: every raised digit limb per ciphertext once per launch, each rotation's key once; writes: both accumulators of
    // every rotation
    const double wk = key_words32 ? 4.0 : 8.0;
    ProfScope ps("inner_product",
                 (src_bytes(src) * batch * lv.ndig * lv.E + (double)rot.n * (wk * 2.0 * lv.ndig * lv.E + 10.0 * lv.E * batch)) * c->N,
                 s);
#define KS_GATHER_LAUNCH(GV, WKT, PK, IS)                                                                                                     \
    hipLaunchKernelGGL((inner_product_kernel<GV, WKT, PK, IS>), dim3(gather_grid(c, lv.E, pl)), dim3(256), 0, s, c->d_mod, lv.ell, lv.E, c->L, \
                       c->M, c->logN, lv.ndig, pl, src, rot, acc)
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
    const GatherTile tile = gather_tile(E, logN, parts_log);
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

// ------------------------------------------------------------------------------------------------
// Several rows of diagonals over the same rotations (the inner sums of a baby-step giant-step transform).  The rotated ciphertext of a
// baby step, sum_j sigma_b(digit_j) key_{b,j} (+ P sigma_b(c0)), is the same for every giant step: a thread forms it once for a slot, reduces
// it and multiplies it by the plaintext slots of `R` giant steps, whose sums it holds.  Keys and gathered slots, which are what
// rotate_mac_kernel reads, are then read once for R sums instead of for each.
//   Four rows of sixteen diagonals, eight ciphertexts, three digits, N = 2^16: 2280 us as four launches of rotate_mac_kernel, 1393; 28 bits
// 1668 -> 768.  What bounds it: the traffic (keys 1.6 GB, plaintexts 1.1, slots), with half of the issue slots.
//   The sums of R = 4 rows take the registers that eight ciphertexts would: a workgroup takes H, up to four, the two halves of a bundle of
// more on the same slots in one workgroup, which so finds keys and plaintexts in cache the second time.  A half's slots of one (position, half of the
// limb) and three digits are 1.8 MB at N = 2^16, which stay in that XCD's L2 from one rotation to the next.
//   Two wavefronts a SIMD do not hide a load of the next step (1684 us): with a set of operands for each digit, up to three, a load has the
// time of a whole rotation.
// ------------------------------------------------------------------------------------------------
// A sum: 64-bit integers for moduli below 2^28 (INT), otherwise mac_wide.
template <bool INT>
struct WideSum {
    double hi;
    uint64_t lo;
    struct Factor {
        double v;
        uint32_t low;
    };
    __device__ __forceinline__ void start(double v) {
        hi = v;
        lo = (uint32_t)__builtin_bit_cast(uint64_t, v + 6755399441055744.0);
    }
    static __device__ __forceinline__ Factor source(uint32_t low, uint32_t top) { return Factor{u64_to_f64((uint64_t)top << 32 | low), low}; }
    template <typename W>
    static __device__ __forceinline__ Factor word(W w) { return Factor{word_to_f64<W>(w), (uint32_t)w}; }
    __device__ __forceinline__ void add(Factor x, Factor k) { mac_wide(x.v, k.v, x.low, k.low, hi, lo); }
    __device__ __forceinline__ Factor reduced(Mod m) const {
        Factor f;
        f.v = mac_wide_reduce(hi, lo, m, &f.low);
        return f;
    }
    __device__ __forceinline__ double result(Mod m) const { return reduce_lazy(reduced(m).v, m); }
};
template <>
struct WideSum<true> {
    int64_t sum;
    using Factor = int32_t;
    __device__ __forceinline__ void start(double v) { sum = (int32_t)v; }
    static __device__ __forceinline__ int32_t source(uint32_t low, uint32_t) { return (int32_t)low; }
    template <typename W>
    static __device__ __forceinline__ int32_t word(W w) { return (int32_t)w; }
    __device__ __forceinline__ void add(int32_t x, int32_t k) { mac_int(x, k, sum); }
    __device__ __forceinline__ int32_t reduced(Mod m) const { return (int32_t)mac_int_reduce(sum, m); }
    __device__ __forceinline__ double result(Mod m) const { return mac_int_reduce(sum, m); }
};
static_assert(kMaxDigits + 1 <= kMacWideTerms && kMacRotations <= kMacWideTerms, "products per sum");

// H of a bundle's `group` ciphertexts, from ciphertext 4 half on.
template <int H>
struct HalfRaw {
    uint32_t lo[H];
    uint32_t hi, from;
};
struct HalfSource {
    BufferRsrc lo, hi;
    uint32_t group, half, hi_bytes;
};
template <int H, bool PACKED>
__device__ __forceinline__ HalfRaw<H> half_load(const HalfSource& src, uint32_t slab, uint32_t N, uint32_t slot) {
    const uint32_t block = slab * N + (__builtin_amdgcn_readfirstlane(slot) & ~63u), lane = threadIdx.x & 63u;
    HalfRaw<H> r;
    r.from = (slot & 63u) * 4;
    buffer_load_words<H>(r.lo, src.lo, lane * (4 * H), block * 4 * src.group + src.half * 1024);
    r.hi = PACKED ? buffer_load<uint32_t>(src.hi, lane * src.hi_bytes & ~3u, block * src.hi_bytes) : 0u;
    return r;
}
template <int H, bool PACKED, bool INT>
__device__ __forceinline__ void half_take(const HalfSource& src, const HalfRaw<H>& l, typename WideSum<INT>::Factor (&x)[H]) {
    uint32_t hi = 0;
    if constexpr (PACKED) hi = from_lane(l.hi >> ((threadIdx.x * src.hi_bytes & 3u) * 8), l.from) >> (16 * src.half);
#pragma unroll
    for (int b = 0; b < H; ++b) x[b] = WideSum<INT>::source(from_lane(l.lo[b], l.from), PACKED ? (hi >> (4 * b)) & 15u : 0u);
}

// 256 threads a half (both in a launch where they have H ciphertexts each); half0: the first of them.
template <int H, int R, typename WK, bool PACKED, bool INT, uint32_t DIGITS>
__global__ __launch_bounds__(512, 2) void rotate_mac_rows_kernel(const Mod* __restrict__ mods, const double* __restrict__ Pmod, uint32_t ell,
                                                                 uint32_t E, uint32_t L, uint32_t M, uint32_t logN, DigitRanges dg,
                                                                 uint32_t parts_log, GatherBundle bundle, MacRotations rot, MacRows rows,
                                                                 uint32_t n_key, uint32_t half0, uint8_t* __restrict__ u,
                                                                 uint64_t u_stride, int accumulate) {
    using Sum = WideSum<INT>;
    using Factor = typename Sum::Factor;
    const uint32_t N = 1u << logN;
    const GatherTile tile = gather_tile(E, logN, parts_log);
    if (!tile.valid) return;  // uniform
    const uint32_t half = half0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), pos = tile.pos, n = tile.n;
    const uint32_t mid = pos < ell ? pos : L + (pos - ell);
    const Mod m = mods[mid];
    const uint64_t slots = ((uint64_t)dg.ndig * E + ell) * N;
    const uint32_t hi_bytes = gather_hi_bytes(bundle.group);
    const HalfSource src{uniform_rsrc(bundle.lo, slots * 4 * bundle.group), uniform_rsrc(bundle.hi, PACKED ? slots * hi_bytes : 0), bundle.group, half, hi_bytes};
    const uint64_t comp = E * packed_limb_bytes(N);
    uint8_t* up = u + (uint64_t)half * 8 * comp + (uint64_t)pos * packed_limb_bytes(N);
    Sum s[R][2 * H];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int b = 0; b < 2 * H; ++b) s[i][b].start(accumulate ? packed_get(up + i * u_stride + b * comp, N, packed_element(n)) : 0.0);
    const Factor pm = [&] {
        const double v = pos < ell ? Pmod[pos] : 0.0;
        return Sum::word((WK)v);
    }();
    struct Raw {
        HalfRaw<H> x;
        WK k0, k1;
    };
    auto fetch = [&](uint32_t r, uint32_t j) {
        Raw w;
        const uint32_t sn = galois_source_slot(n, rot.galois[r], logN);
        // a key is below 4 GB: [8][2][255][2^16] words of at most 8 bytes
        const BufferRsrc key = uniform_rsrc(rot.key[r], (uint64_t)dg.ndig * 2 * M * N * sizeof(WK));
        const uint32_t at = (j * 2 * M + mid) * N * (uint32_t)sizeof(WK);
        w.x = half_load<H, PACKED>(src, j * E + pos, N, sn);
        w.k0 = buffer_load<WK>(key, n * (uint32_t)sizeof(WK), at);
        w.k1 = buffer_load<WK>(key, n * (uint32_t)sizeof(WK), at + M * N * (uint32_t)sizeof(WK));
        return w;
    };
    const auto plaintexts = [&](uint32_t r, WK (&w)[R]) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const void* pt = rows.pt[i][r];   // uniform; null: the constant 1
            w[i] = pt ? buffer_load<WK>(uniform_rsrc(pt, (uint64_t)M * N * sizeof(WK)), n * (uint32_t)sizeof(WK), mid * N * (uint32_t)sizeof(WK)) : (WK)1;
        }
    };
    // One rotation after the other.  DIGITS: what a step has used is requested again for the next rotation, so that a load has a whole
    // rotation to arrive; 0: any number of digits, one step ahead.
    if (n_key != 0) {   // uniform
        constexpr uint32_t SETS = DIGITS ? DIGITS : 1;
        Raw set[SETS];
#pragma unroll
        for (uint32_t j = 0; j < SETS; ++j) set[j] = fetch(0, j);
#pragma unroll 1
        for (uint32_t r = 0; r < n_key; ++r) {
            const uint32_t after = min(r + 1, n_key - 1);
            WK w[R];
            plaintexts(r, w);
            // (above ell the addend's slabs have none for this position: any other is read against a factor of zero)
            const HalfRaw<H> c0 = half_load<H, PACKED>(src, dg.ndig * E + min(pos, ell - 1), N, galois_source_slot(n, rot.galois[r], logN));
            Sum t[2 * H];
#pragma unroll
            for (int b = 0; b < 2 * H; ++b) t[b].start(0.0);
            const auto step = [&](const Raw& q) {
                __builtin_amdgcn_sched_barrier(0);
                const Factor k0 = Sum::word(q.k0), k1 = Sum::word(q.k1);
                Factor x[H];
                half_take<H, PACKED, INT>(src, q.x, x);
#pragma unroll
                for (int b = 0; b < H; ++b) {
                    t[2 * b].add(x[b], k0);
                    t[2 * b + 1].add(x[b], k1);
                }
            };
            if constexpr (DIGITS != 0) {
#pragma unroll
                for (uint32_t j = 0; j < DIGITS; ++j) {
                    step(set[j]);
                    set[j] = fetch(after, j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll 1
                for (uint32_t j = 0; j < dg.ndig; ++j) {
                    const bool last = j + 1 == dg.ndig;
                    const Raw next = fetch(last ? after : r, last ? 0 : j + 1);
                    step(set[0]);
                    set[0] = next;
                }
            }
            Factor x[H];
            half_take<H, PACKED, INT>(src, c0, x);
#pragma unroll
            for (int b = 0; b < H; ++b) t[2 * b].add(x[b], pm);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < 2 * H; ++b) {
                const Factor v = t[b].reduced(m);
#pragma unroll
                for (int i = 0; i < R; ++i) s[i][b].add(v, Sum::word(w[i]));
                __builtin_amdgcn_sched_barrier(0);   // one at a time: the registers are taken
            }
        }
    }
    if (pos < ell) {  // uniform: P (c0, c1) of the identities
        uint32_t own = 0;
        while (own + 1 < dg.ndig && pos >= dg.hi[own]) ++own;
#pragma unroll 1
        for (uint32_t r = n_key; r < rot.n; ++r) {
            WK w[R];
            plaintexts(r, w);
            const HalfRaw<H> r0 = half_load<H, PACKED>(src, dg.ndig * E + pos, N, n), r1 = half_load<H, PACKED>(src, own * E + pos, N, n);
            Factor x[2][H];
            half_take<H, PACKED, INT>(src, r0, x[0]);
            half_take<H, PACKED, INT>(src, r1, x[1]);
#pragma unroll
            for (int b = 0; b < 2 * H; ++b) {
                Sum t;
                t.start(0.0);
                t.add(x[b & 1][b / 2], pm);
                const Factor v = t.reduced(m);
#pragma unroll
                for (int i = 0; i < R; ++i) s[i][b].add(v, Sum::word(w[i]));
            }
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        double sums[2 * H];
#pragma unroll
        for (int b = 0; b < 2 * H; ++b) sums[b] = s[i][b].result(m);
        packed_put<2 * H>(up + i * u_stride, comp, N, packed_element(n & ~63u), sums);
    }
}

void launch_rotate_mac_rows(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, const MacRows& rows, uint8_t* u,
                            uint64_t u_stride, bool accumulate, hipStream_t s, bool key_words32) {
    if (rot.n == 0) return;
    // quarters where the slots of a half are more than an XCD's L2 keeps beside the streams: eight ciphertexts, N = 2^16, three digits (3.5 MB)
    // 1472 -> 1393 us; two digits (2.4 MB) 1350 -> 1336, 28 bits (3.1 MB) 768 -> 790, two ciphertexts 669 -> 677
    const bool large = lv.ndig * src.group * src_bytes(src) * (c->N / 2) > 3.3 * (1 << 20);
    const uint32_t pl = std::max(gather_parts_log(lv.E), large ? 2u : 1u);
    DigitRanges dg;
    dg.ndig = lv.ndig;
    for (uint32_t j = 0; j < kMaxDigits; ++j) {
        dg.lo[j] = j < lv.ndig ? lv.digit_lo[j] : 0;
        dg.hi[j] = j < lv.ndig ? lv.digit_hi[j] : 0;
    }
    MacRotations sorted = rot;
    MacRows pts = rows;
    uint32_t n_key = 0, n_id = 0;
    for (int pass = 0; pass < 2; ++pass)
        for (uint32_t r = 0; r < rot.n; ++r) {
            if ((rot.galois[r] == 1) != (pass == 1)) continue;
            const uint32_t to = n_key + n_id;
            sorted.galois[to] = rot.galois[r];
            sorted.key[to] = rot.key[r];
            for (uint32_t i = 0; i < rows.n; ++i) pts.pt[i][to] = rows.pt[i][r];
            ++(pass == 0 ? n_key : n_id);
        }
    // reads and writes as rotate_mac's, but one pass over slots and keys for all rows
    const double wk = key_words32 ? 4.0 : 8.0;
    const double reads = src.group * src_bytes(src) * (lv.ndig * lv.E + lv.ell) + wk * (double)rot.n * (2.0 * lv.ndig + rows.n) * lv.E;
    ProfScope ps("rotate_mac_rows", (reads + (double)src.group * 10 * lv.E * rows.n * (accumulate ? 2 : 1)) * c->N, s,
                 (double)rot.n * lv.E * c->N * 4.0 * src.group * (2 * lv.ndig + 1 + 2 * rows.n));
    const bool words32 = !src.hi, ints = words32 && integer_sums(c);
    const auto launch = [&](uint32_t h, uint32_t half0, uint32_t n_halves) {
        const dim3 grid(gather_grid(c, lv.E, pl)), block(256 * n_halves);
#define KS_LAUNCH_ROWS(HV, RV, WKT, PK, IS, DG)                                                                                                \
    hipLaunchKernelGGL((rotate_mac_rows_kernel<HV, RV, WKT, PK, IS, DG>), grid, block, 0, s, c->d_mod, c->d_Pmod, lv.ell, lv.E, c->L, c->M,     \
                       c->logN, dg, pl, src, sorted, pts, n_key, half0, u, u_stride, accumulate ? 1 : 0)
#define KS_LAUNCH_R(HV, WKT, PK, IS)                                                              \
    if (rows.n != kMacRows) KS_LAUNCH_ROWS(HV, 2, WKT, PK, IS, 0);                                \
    else if (HV == 4 && lv.ndig == 1) KS_LAUNCH_ROWS(HV, kMacRows, WKT, PK, IS, HV == 4 ? 1 : 0); \
    else if (HV == 4 && lv.ndig == 2) KS_LAUNCH_ROWS(HV, kMacRows, WKT, PK, IS, HV == 4 ? 2 : 0); \
    else if (HV == 4 && lv.ndig == 3) KS_LAUNCH_ROWS(HV, kMacRows, WKT, PK, IS, HV == 4 ? 3 : 0); \
    else KS_LAUNCH_ROWS(HV, kMacRows, WKT, PK, IS, 0)
#define KS_LAUNCH_H(HV)                                              \
    {                                                                \
        if (ints) { KS_LAUNCH_R(HV, uint32_t, false, true); }        \
        else if (words32) { KS_LAUNCH_R(HV, uint32_t, false, false); } \
        else { KS_LAUNCH_R(HV, uint64_t, true, false); }             \
    }
        switch (h) {
            case 1: KS_LAUNCH_H(1) break;
            case 2: KS_LAUNCH_H(2) break;
            case 3: KS_LAUNCH_H(3) break;
            default: KS_LAUNCH_H(4) break;
        }
#undef KS_LAUNCH_H
#undef KS_LAUNCH_R
#undef KS_LAUNCH_ROWS
    };
    if (src.group <= 4) launch(src.group, 0, 1);
    else if (src.group == 8) launch(4, 0, 2);
    else {
        launch(4, 0, 1);
        launch(src.group - 4, 1, 1);
    }
}

}  // namespace ks
