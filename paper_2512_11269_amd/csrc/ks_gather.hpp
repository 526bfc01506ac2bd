// What the gather kernels share: a bundle's slots, sums of products, the order of the workgroups.
#pragma once
#include "ks_internal.hpp"
#include "ks_tiles.hpp"

namespace ks {

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
// every rotation but the first finds its sources in that L2.  parts_log: gather_parts_log; thread: 0 .. 255.
struct GatherTile {
    uint32_t pos, n;
    bool valid;
};
__device__ __forceinline__ GatherTile gather_tile(uint32_t E, uint32_t logN, uint32_t parts_log, uint32_t thread) {
    const uint32_t per_unit = 1u << (logN - 8 - parts_log), local = blockIdx.x >> 3;
    const uint32_t unit = (local / per_unit) * 8 + (blockIdx.x & 7);
    GatherTile t;
    t.valid = unit < (E << parts_log);
    t.pos = unit >> parts_log;
    t.n = (((unit & ((1u << parts_log) - 1)) * per_unit + local % per_unit) << 8) + thread;
    return t;
}
inline uint32_t gather_grid(const ks_ctx* c, uint32_t E, uint32_t parts_log) {
    return (((E << parts_log) + 7) / 8) * 8 * ((c->N / 256) >> parts_log);
}

// Integer sums: every modulus below 2^28 (250 products of a residue and a lazy one, 0.51 * 2^56 each, stay below 2^63).
// Eight ciphertexts, N = 2^16, E = 32, three digits, fp64 -> integer sums: calls of 16 rotations multiplied and summed 960 -> 869 us
// (82 registers instead of 134); at 28 bits no size was slower.
inline bool integer_sums(const ks_ctx* c) {
    for (uint64_t m : c->mod)
        if (m >> 28) return false;
    return true;
}
// bytes a gathered source residue takes
inline double src_bytes(const GatherBundle& g) { return g.hi ? 4.0 + (double)gather_hi_bytes(g.group) / g.group : 4.0; }

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

}  // namespace ks
