// Tile-level pieces of the two-phase transform, shared by the plain NTT kernels and the fused ones.
//
// A limb is an R x 256 matrix (R = N / 256 = 16 .. 256).  "Row" pieces work on contiguous 256-point rows, one
// wavefront owning four rows (16 lanes per row, 16 points per lane); "column" pieces work on a tile of 4096 / R
// columns x R rows (16 x 256 for N = 2^16) owned by a 256-thread workgroup.  Twiddles come from the per-modulus heap-ordered
// table W[k] = psi^brv(k): the forward stage with 2^s blocks uses W[2^s + block].
#pragma once
#include "ks_device.hpp"

namespace ks {

// Digit partition handed to kernels by value.
struct DigitRanges {
    uint32_t ndig;
    uint32_t lo[8], hi[8];
};

// log2 of the parts into which the rotation gathers cut each of the E limb positions (gather_tile).  Halves keep a part's
// sources to one XCD's L2; where E % 4 is 1 or 2, halves leave 6 or 4 of the eight XCDs idle in the last round, and quarters
// pay for sources that two XCDs then read (eighths only in few rounds).  Sixteen rotation-multiplications of eight
// ciphertexts, N = 2^16, halves -> quarters: E = 10 226 -> 212 us, 17 566 -> 553, 26 1050 -> 1026, but 12 268 -> 271,
// 23 730 -> 738, 32 1274 -> 1288; E = 9 in eighths 207 -> 189, quarters 193; 13 -4.6 and -5.4 %, at N = 2^14 +3.8 and -1.3 %.
constexpr uint32_t gather_parts_log(uint32_t E) { return E % 4 == 1 ? (E < 12 ? 3 : 2) : E % 4 == 2 ? 2 : 1; }

// Slot permutation of sigma_g (X -> X^g) on a bit-reversed evaluation vector: slot n holds the point
// psi^(2 brv(n) + 1); sigma_g(a) evaluated there is a evaluated at that point raised to g.
__device__ __forceinline__ uint32_t galois_source_slot(uint32_t n, uint32_t g, uint32_t logN) {
    // both factors are below 2^17: the full-rate 24-bit product has the bits that count
    const uint32_t e = __umul24(g, 2u * (__brev(n) >> (32 - logN)) + 1u) & ((2u << logN) - 1u);
    return __brev((e - 1u) >> 1) >> (32 - logN);
}

constexpr int kRowPitch = 272;  // 256 points + 1 pad per 16: the transposed LDS accesses hit distinct banks


// Twiddles of the two register passes of a tile core, loaded ahead of the butterflies.
struct PassTwiddles {
    double a[16], b[16];
};
// One direction's twiddle tables (device pointers, every table indexed [modulus id][...]):
//   W    [N]     W[k] = psi^brv(k) (or psi^-brv(k)), heap order
//   trow [N/16]  trow[i] = W[8 (N/16 + i)] = psi^(1 + 2 brv(i)): the generator of the last register pass of row-pass lane i
//   w16  [8]     w16[e] = omega^e, omega = psi^(N/8) a primitive 16th root of unity
struct TwTables {
    const double* W;
    const double* trow;
    const double* w16;
};

// rows: node = R + row; lane j0 owns points 16 j0 .. 16 j0 + 15 in the second pass.
// The second pass needs the 15 table entries below heap node n = 16 node + j0 -- one twiddle per point of the row,
// as much data as the row itself.  They factor as W[n 2^u + g] = T^(2^(3-u)) * omega^(2^(3-u) brv_u(g)) with
// T = W[8 n], so one load, three squarings and eleven products replace fifteen loads (row kernels are
// bandwidth-bound and have arithmetic to spare).
__device__ __forceinline__ void load_row_twiddles_b(double (&tb)[16], const TwTables& tbl, uint32_t mod_id, uint32_t N, uint32_t node,
                                                    uint32_t j0, Mod m) {
    const double* w = tbl.w16 + mod_id * 8;
    const double T1 = tbl.trow[(size_t)mod_id * (N / 16) + (node * 16 + j0 - N / 16)];
    const double T2 = mulmod_lazy(T1, T1, m), T4 = mulmod_lazy(T2, T2, m), T8 = mulmod_lazy(T4, T4, m);
    tb[0] = 0.0;
    tb[1] = T8;
    tb[2] = T4;  tb[3] = mulmod_lazy(T4, w[4], m);
    tb[4] = T2;  tb[5] = mulmod_lazy(T2, w[4], m);  tb[6] = mulmod_lazy(T2, w[2], m);  tb[7] = mulmod_lazy(T2, w[6], m);
    tb[8] = T1;  tb[9] = mulmod_lazy(T1, w[4], m);  tb[10] = mulmod_lazy(T1, w[2], m); tb[11] = mulmod_lazy(T1, w[6], m);
    tb[12] = mulmod_lazy(T1, w[1], m);  tb[13] = mulmod_lazy(T1, w[5], m);
    tb[14] = mulmod_lazy(T1, w[3], m);  tb[15] = mulmod_lazy(T1, w[7], m);
}
// Both passes (kernels that keep the first one's in LDS: row_twiddles_to_lds).
__device__ __forceinline__ void load_row_twiddles(PassTwiddles& t, const TwTables& tbl, uint32_t mod_id, uint32_t N, uint32_t node,
                                                  uint32_t j0, Mod m) {
    load_twiddles16(t.a, tbl.W + (size_t)mod_id * N, node);
    load_row_twiddles_b(t.b, tbl, mod_id, N, node, j0, m);
}
// First-pass twiddles of a row (the 15 table entries below heap node `node`, the same for the row's 16 lanes) placed in
// 16 doubles of LDS: lane j0 fetches entry j0.  Frees 30 registers per lane where a kernel is short of them; the
// butterflies then read them as LDS broadcasts.  The caller synchronises before use.
__device__ __forceinline__ void row_twiddles_to_lds(double* ta_row, const double* __restrict__ W, uint32_t node, uint32_t j0) {
    const uint32_t u = 31u - __clz(j0 | 1u), g = j0 - (1u << u);
    ta_row[j0] = j0 ? W[(node << u) + g] : 0.0;
}

// Both passes' twiddles of a wavefront's four rows in LDS, for a kernel that uses them again and again: entry k of the first pass at
// ta[16 (lane / 16) + k], of the second (load_row_twiddles' t.b) at tb[64 (k - 1) + lane].  The caller synchronises before use.
__device__ __forceinline__ void store_row_twiddles(double* ta, double* tb, const TwTables& tbl, uint32_t mod_id, uint32_t N, uint32_t node,
                                                   uint32_t lane, Mod m) {
    row_twiddles_to_lds(ta + (lane >> 4) * 16, tbl.W + (size_t)mod_id * N, node, lane & 15u);
    double t[16];
    load_row_twiddles_b(t, tbl, mod_id, N, node, lane & 15u, m);
#pragma unroll
    for (int k = 1; k < 16; ++k) tb[64 * (k - 1) + lane] = t[k];
}

// Columns (R = 2^LOG_R rows, 4 <= LOG_R <= 8): the first register pass runs global stages 0..3 with the sub-tree below
// heap node 1; the second one the remaining E = LOG_R - 4 stages on 16 consecutive rows 16 r0 + k, as the last E local
// stages of a 16-point pass: local stage ul = 4 - E + u is global stage 4 + u, whose block of row 16 r0 + k is
// r0 2^ul + (k >> (4 - ul)), so its table entry (1 << ul) + g holds W[2^(E + ul) + r0 2^ul + g].  For E = 4 that is
// the sub-tree below node 16 + r0.
template <int LOG_R>
__device__ __forceinline__ void load_col_twiddles(PassTwiddles& t, const double* __restrict__ W, uint32_t r0) {
    constexpr int E = LOG_R - 4;
    load_twiddles16(t.a, W, 1);
    if constexpr (E > 0) {
#pragma unroll
        for (int ul = 4 - E; ul < 4; ++ul)
#pragma unroll
            for (int g = 0; g < (1 << ul); ++g) t.b[(1 << ul) + g] = W[(1u << (E + ul)) + (r0 << ul) + g];
    }
}

// Last 8 forward stages of one row.  in: v[k] = point j0 + 16 k of the row, lazy with |v| <= 8 p.
// out: v[k] = transformed point j0 + 16 k, lazy with |v| <= |in| + 4.1 p.
// lrow: this row's kRowPitch doubles of LDS, shared by the row's 16 lanes (all in one wavefront).
__device__ __forceinline__ void row_fwd_core(double (&v)[16], const PassTwiddles& t, uint32_t j0, double* lrow, Mod m) {
    radix16_fwd(v, t.a, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) lrow[j0 + 17 * k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = lrow[17 * j0 + k];
    radix16_fwd(v, t.b, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) lrow[17 * j0 + k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = lrow[j0 + 17 * k];
}

// The same without the last exchange: out v[k] = point 16 j0 + k (sixteen consecutive points per thread).
__device__ __forceinline__ void row_fwd_core_consecutive(double (&v)[16], const PassTwiddles& t, uint32_t j0, double* lrow, Mod m) {
    radix16_fwd(v, t.a, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) lrow[j0 + 17 * k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = lrow[17 * j0 + k];
    radix16_fwd(v, t.b, m);
}

// radix16_fwd with twiddles from LDS (t[stride * k], k = 1..15), fenced stage by stage so that no more than a stage's are in
// registers at a time.
template <int U = 0>
__device__ __forceinline__ void radix16_fwd_lds(double (&v)[16], const double* t, uint32_t stride, Mod m) {
    constexpr int HALF = 8 >> U;
    double w[1 << U];
#pragma unroll
    for (int g = 0; g < (1 << U); ++g) w[g] = t[stride * ((1 << U) + g)];
#pragma unroll
    for (int g = 0; g < (1 << U); ++g)
#pragma unroll
        for (int i = 0; i < HALF; ++i) {
            const int k = g * 2 * HALF + i;
            const double x = mulmod_lazy(v[k + HALF], w[g], m);
            v[k + HALF] = v[k] - x;
            v[k] = v[k] + x;
        }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (U < 3) radix16_fwd_lds<U + 1>(v, t, stride, m);
}
// radix16_inv the same way.
template <int U = 3>
__device__ __forceinline__ void radix16_inv_lds(double (&v)[16], const double* t, uint32_t stride, Mod m) {
    constexpr int HALF = 8 >> U;
    double w[1 << U];
#pragma unroll
    for (int g = 0; g < (1 << U); ++g) w[g] = t[stride * ((1 << U) + g)];
#pragma unroll
    for (int g = 0; g < (1 << U); ++g)
#pragma unroll
        for (int i = 0; i < HALF; ++i) {
            const int k = g * 2 * HALF + i;
            const double x = v[k], y = v[k + HALF];
            v[k] = x + y;
            v[k + HALF] = mulmod_lazy(x - y, w[g], m);
        }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (U > 0) radix16_inv_lds<U - 1>(v, t, stride, m);
}
// What a wavefront wrote to LDS can be read by its other lanes (LDS takes a wavefront's accesses in order; this keeps the compiler to it).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// First 8 inverse stages of one row (t built from the inverse table).  in: v[k] = point j0 + 16 k, |v| <= p.
// out: same layout, |v| <= 0.51 p.
__device__ __forceinline__ void row_inv_core(double (&v)[16], const PassTwiddles& t, uint32_t j0, double* lrow, Mod m) {
#pragma unroll
    for (int k = 0; k < 16; ++k) lrow[j0 + 17 * k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = lrow[17 * j0 + k];
    radix16_inv(v, t.b, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) lrow[17 * j0 + k] = reduce_lazy(v[k], m);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = lrow[j0 + 17 * k];
    radix16_inv(v, t.a, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = reduce_lazy(v[k], m);
}

// First log2(R) forward stages on a column tile of TC columns x R rows (R = 2^LOG_R), TC R / 16 threads, thread
// (c = tid % TC, r0 = tid / TC).  in: v[k] = row r0 + (R / 16) k; out: v[k] = row 16 r0 + k; lds: R TC doubles (unused for
// R = 16, where one register pass does everything and rows k go in and out).  Growth: at most 0.51 p per stage.
template <int LOG_R, int TC = (4096 >> LOG_R)>
__device__ __forceinline__ void col_fwd_core(double (&v)[16], const PassTwiddles& t, uint32_t c, uint32_t r0, double* lds, Mod m) {
    constexpr int E = LOG_R - 4, S = 1 << E;
    radix16_fwd(v, t.a, m);
    if constexpr (E > 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) lds[(r0 + S * k) * TC + c] = v[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = lds[(16 * r0 + k) * TC + c];
        radix16_fwd<4 - E>(v, t.b, m);
    }
}

// Last log2(R) inverse stages on a column tile (no N^-1 factor): in rows 16 r0 + k, out rows r0 + (R / 16) k.
// in: |v| <= p.  out: |v| <= 16 p.
template <int LOG_R, int TC = (4096 >> LOG_R)>
__device__ __forceinline__ void col_inv_core(double (&v)[16], const PassTwiddles& t, uint32_t c, uint32_t r0, double* lds, Mod m) {
    constexpr int E = LOG_R - 4, S = 1 << E;
    if constexpr (E > 0) {
        radix16_inv<4 - E>(v, t.b, m);
#pragma unroll
        for (int k = 0; k < 16; ++k) lds[(16 * r0 + k) * TC + c] = reduce_lazy(v[k], m);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = lds[(r0 + S * k) * TC + c];
    }
    radix16_inv(v, t.a, m);
}

// Buffer descriptor of a tensor slice (raw, unstrided; gfx9 data-format word): loads through it take a per-lane byte
// offset in a vector register plus a uniform byte offset in a scalar register, and reads beyond `bytes` return zero.
using BufferRsrc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ BufferRsrc make_buffer_rsrc(const void* base, uint64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(uint32_t)bytes, 0x00020000);
}

// ---- packed limbs ----------------------------------------------------------------------------------------------------
// Between its kernels a call keeps a limb as N 32-bit low words followed by N bytes, 5 bytes a residue instead of 8: a value v
// (|v| < 2^39: every lazy representative of the chain, unreduced) is stored as the 40 bits of v + 2^39.  Packing is one addition and
// a byte permutation, unpacking the reverse.
//   Elements are ordered for the kernels at both ends, which move 16 values a thread: element 4 (256 g + j) + x is word x of
// the 16 bytes `j` of a group g of four rows, and byte x of the 4 bytes `j`.  A thread takes four accesses of 16 and four of 4 bytes,
// each of them contiguous over a wavefront, where 8-byte rows took sixteen.  What the element is depends on the two ends:
//   rows -> rows  (accumulators, tensor product): j = 64 i + lane, value k = 4 i + x of that lane: row lane / 16, column lane % 16 + 16 k;
//   rows <-> columns (half-transformed limbs): j is the column and x the row.  A row thread holds 16 columns of one row and a
// column thread 16 rows of one column, so the row kernels exchange blocks of 4 x 4 among the lanes that share a column group
// (exchange_rows: one instruction a value, no LDS);
//   columns -> conversion (sources, see load_source): j is the column, row x of group 4 r0 + q the strided row r0 + (R / 16) (4 q + x):
// the values that one thread leaves and one thread of the conversion takes.
constexpr double kPackBias = 0x1.8p52 + 0x1p39;
KS_HD constexpr uint64_t packed_limb_bytes(uint64_t N) { return 5 * N; }

struct alignas(16) Words4 {
    uint32_t w[4];
};
struct PackedRaw {
    uint32_t lo[16], hi[4];
};
// The lowest bytes of four words.
__device__ __forceinline__ uint32_t low_bytes(uint32_t h0, uint32_t h1, uint32_t h2, uint32_t h3) {
    return __builtin_amdgcn_perm(h1, h0, 0x0c0c0400) | __builtin_amdgcn_perm(h3, h2, 0x04000c0c);
}
// at: 256 g + lane with STEP 64 (rows), 1024 r0 + column with STEP 256 (columns)
template <uint32_t STEP>
__device__ __forceinline__ PackedRaw packed_load(const uint8_t* limb, uint32_t N, uint32_t at) {
    const Words4* lo = reinterpret_cast<const Words4*>(limb) + at;
    const uint32_t* hi = reinterpret_cast<const uint32_t*>(limb + 4 * (size_t)N) + at;
    PackedRaw r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const Words4 q = lo[i * STEP];
#pragma unroll
        for (int x = 0; x < 4; ++x) r.lo[4 * i + x] = q.w[x];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) r.hi[i] = hi[i * STEP];
    return r;
}
template <uint32_t STEP>
__device__ __forceinline__ void packed_store(uint8_t* limb, uint32_t N, uint32_t at, const PackedRaw& r) {
    Words4* lo = reinterpret_cast<Words4*>(limb) + at;
    uint32_t* hi = reinterpret_cast<uint32_t*>(limb + 4 * (size_t)N) + at;
#pragma unroll
    for (int i = 0; i < 4; ++i) lo[i * STEP] = Words4{{r.lo[4 * i], r.lo[4 * i + 1], r.lo[4 * i + 2], r.lo[4 * i + 3]}};
#pragma unroll
    for (int i = 0; i < 4; ++i) hi[i * STEP] = r.hi[i];
}
// Columns order inside a limb of 64-bit words, for transforms in place: a tile of TC columns keeps to the bytes of its own columns.  Of
// the four rows of a group the low words take the first two, 16 bytes a column, and the bytes above half of the third.
struct InPlaceOffsets {
    uint32_t lo, hi;
};
template <int TC>
__device__ __forceinline__ InPlaceOffsets in_place_offsets(uint32_t col) {
    const uint32_t c = col % TC, tile = (col - c) * 8;
    return InPlaceOffsets{c / (TC / 2) * 2048 + tile + c % (TC / 2) * 16, 4096 + tile + c * 4};
}
constexpr uint32_t kQuadBytes = 8192;   // four rows of 256 words
// rows: lane of group rg; columns: group q of thread (r0, column)
template <int TC>
__device__ __forceinline__ PackedRaw in_place_load_rows(const uint64_t* limb, uint32_t rg, uint32_t lane) {
    const uint8_t* group = reinterpret_cast<const uint8_t*>(limb) + rg * kQuadBytes;
    PackedRaw r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const InPlaceOffsets o = in_place_offsets<TC>(64 * i + lane);
        const Words4 w = *reinterpret_cast<const Words4*>(group + o.lo);
#pragma unroll
        for (int x = 0; x < 4; ++x) r.lo[4 * i + x] = w.w[x];
        r.hi[i] = *reinterpret_cast<const uint32_t*>(group + o.hi);
    }
    return r;
}
template <int TC>
__device__ __forceinline__ void in_place_store_rows(uint64_t* limb, uint32_t rg, uint32_t lane, const PackedRaw& r) {
    uint8_t* group = reinterpret_cast<uint8_t*>(limb) + rg * kQuadBytes;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const InPlaceOffsets o = in_place_offsets<TC>(64 * i + lane);
        *reinterpret_cast<Words4*>(group + o.lo) = Words4{{r.lo[4 * i], r.lo[4 * i + 1], r.lo[4 * i + 2], r.lo[4 * i + 3]}};
        *reinterpret_cast<uint32_t*>(group + o.hi) = r.hi[i];
    }
}
template <int TC>
__device__ __forceinline__ PackedRaw in_place_load_cols(const uint64_t* limb, uint32_t r0, uint32_t col) {
    const InPlaceOffsets o = in_place_offsets<TC>(col);
    const uint8_t* group = reinterpret_cast<const uint8_t*>(limb) + r0 * (4 * kQuadBytes);
    PackedRaw r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const Words4 w = *reinterpret_cast<const Words4*>(group + q * kQuadBytes + o.lo);
#pragma unroll
        for (int x = 0; x < 4; ++x) r.lo[4 * q + x] = w.w[x];
        r.hi[q] = *reinterpret_cast<const uint32_t*>(group + q * kQuadBytes + o.hi);
    }
    return r;
}
template <int TC>
__device__ __forceinline__ void in_place_store_cols(uint64_t* limb, uint32_t r0, uint32_t col, const PackedRaw& r) {
    const InPlaceOffsets o = in_place_offsets<TC>(col);
    uint8_t* group = reinterpret_cast<uint8_t*>(limb) + r0 * (4 * kQuadBytes);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        *reinterpret_cast<Words4*>(group + q * kQuadBytes + o.lo) = Words4{{r.lo[4 * q], r.lo[4 * q + 1], r.lo[4 * q + 2], r.lo[4 * q + 3]}};
        *reinterpret_cast<uint32_t*>(group + q * kQuadBytes + o.hi) = r.hi[q];
    }
}
// N = 2^12 has no exchange through LDS between a column tile's loads and its stores: everything has arrived before anything is
// overwritten.
template <int LOG_R>
__device__ __forceinline__ void tile_loaded(double (&v)[16]) {
    if constexpr (LOG_R == 4) {
#pragma unroll
        for (int k = 0; k < 16; ++k) asm volatile("" : "+v"(v[k]));
        __syncthreads();
    }
}

// Kernels with one thread per slot: 64 consecutive slots are 64 consecutive elements in the rows -> rows order, permuted.
__device__ __forceinline__ uint32_t packed_element(uint32_t n) {
    return (n & ~1023u) | (n & 192u) << 2 | (n & 768u) >> 2 | (n & 15u) << 2 | ((n >> 4) & 3u);
}
__device__ __forceinline__ double packed_get(const uint8_t* limb, uint32_t N, uint32_t e) {
    const uint64_t bits = (uint64_t)(0x43380000u | limb[4 * (size_t)N + e]) << 32 | reinterpret_cast<const uint32_t*>(limb)[e];
    return __builtin_bit_cast(double, bits) - kPackBias;
}

// The values of slot n of LIMBS limbs stored by a wavefront that holds 64 consecutive slots: the lanes exchange what they hold, so that
// a lane's neighbours write its neighbours in memory (as permuted stores every 16 lanes touch four times the lines: four rotations of
// eight ciphertexts, N = 2^16, 315 -> 413 us).  limb: the first of the limbs, `stride` bytes apart; element: packed_element of the
// wavefront's first slot.
template <int LIMBS>
__device__ __forceinline__ void packed_put(uint8_t* limb, uint64_t stride, uint32_t N, uint32_t element, const double (&v)[LIMBS]) {
    const uint32_t lane = threadIdx.x & 63u, from = ((lane & 3u) * 16 + (lane >> 2)) * 4, e = element + lane;
    uint32_t h[(LIMBS + 3) / 4 * 4] = {};
#pragma unroll
    for (int i = 0; i < LIMBS; ++i) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, v[i] + kPackBias);
        reinterpret_cast<uint32_t*>(limb + i * stride)[e] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)from, (int)(uint32_t)bits);
        h[i] = (uint32_t)(bits >> 32);
    }
#pragma unroll
    for (int i = 0; i < LIMBS; i += 4) {
        const uint32_t b = (uint32_t)__builtin_amdgcn_ds_bpermute((int)from, (int)low_bytes(h[i], h[i + 1], h[i + 2], h[i + 3]));
#pragma unroll
        for (int x = 0; x < 4 && i + x < LIMBS; ++x) (limb + (i + x) * stride)[4 * (size_t)N + e] = (uint8_t)(b >> (8 * x));
    }
}

// Byte x of every word -> word x: r[i] byte x becomes r[x] byte i.
__device__ __forceinline__ void transpose_bytes(uint32_t (&r)[4]) {
    const uint32_t a = __builtin_amdgcn_perm(r[1], r[0], 0x05010400), b = __builtin_amdgcn_perm(r[3], r[2], 0x05010400);
    const uint32_t c = __builtin_amdgcn_perm(r[1], r[0], 0x07030602), d = __builtin_amdgcn_perm(r[3], r[2], 0x07030602);
    r[0] = __builtin_amdgcn_perm(b, a, 0x05040100);
    r[1] = __builtin_amdgcn_perm(b, a, 0x07060302);
    r[2] = __builtin_amdgcn_perm(d, c, 0x05040100);
    r[3] = __builtin_amdgcn_perm(d, c, 0x07060302);
}
// Word x of lane l + 16 i becomes word i of lane l + 16 x (l < 16): a 4 x 4 transposition, its own inverse.
__device__ __forceinline__ void exchange_rows(uint32_t* r) {
    const auto a = __builtin_amdgcn_permlane32_swap(r[0], r[2], false, false), b = __builtin_amdgcn_permlane32_swap(r[1], r[3], false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false), d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    r[0] = c[0];
    r[1] = c[1];
    r[2] = d[0];
    r[3] = d[1];
}
// Sixteen values of a thread, in the order of their elements: byte x of hi[i] goes with lo[4 i + x].
__device__ __forceinline__ PackedRaw pack(const double (&v)[16], double bias = kPackBias) {
    PackedRaw r;
    uint32_t h[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, v[k] + bias);
        r.lo[k] = (uint32_t)bits;
        h[k] = (uint32_t)(bits >> 32);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) r.hi[i] = low_bytes(h[4 * i], h[4 * i + 1], h[4 * i + 2], h[4 * i + 3]);
    return r;
}
__device__ __forceinline__ double unpack_one(uint32_t lo, uint32_t bytes, int x) {
    const uint32_t hi = __builtin_amdgcn_perm(0x43380000u, bytes, 0x07060500u + x);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo) - kPackBias;
}
__device__ __forceinline__ void unpack(const PackedRaw& r, double (&v)[16]) {
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = unpack_one(r.lo[k], r.hi[k >> 2], k & 3);
}
// The same for a row thread whose limb is in columns order: value k is column 16 k + lane % 16 of the thread's row, and the element
// that a lane loads or stores belongs to row x of column 64 i + lane.
__device__ __forceinline__ PackedRaw pack_rows(const double (&v)[16]) {
    PackedRaw r;
    uint32_t h[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, v[k] + kPackBias);
        r.lo[k] = (uint32_t)bits;
        h[k] = (uint32_t)(bits >> 32);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) exchange_rows(r.lo + 4 * i);
#pragma unroll
    for (int x = 0; x < 4; ++x) r.hi[x] = low_bytes(h[x], h[4 + x], h[8 + x], h[12 + x]);
    exchange_rows(r.hi);
    transpose_bytes(r.hi);
    return r;
}
__device__ __forceinline__ void unpack_rows(PackedRaw r, double (&v)[16]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) exchange_rows(r.lo + 4 * i);
    transpose_bytes(r.hi);
    exchange_rows(r.hi);
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = unpack_one(r.lo[k], r.hi[k & 3], k >> 2);
}

// Sources of a conversion: y + 0x80808080 of a residue |y| < 2^36 (canonical, or the signed remainder of a rescale) as the low
// word and the (signed) byte above.  With the top bit of each byte flipped the word is the residue's signed base-256 digits
// d_0..d_3 (digit = byte - 128), and the byte is d_4, |d_4| <= 17.  The bytes of a thread's 16 values are 16 consecutive ones,
// inside the 64 bytes of a group of rows that a column tile of 16 owns (the limb is converted in place, tile by tile).
constexpr double kDigitBias = 6755399441055744.0 + 2155905152.0;   // 1.5 * 2^52 + 0x80808080
__device__ __forceinline__ uint32_t source_bytes_offset(uint32_t r0, uint32_t col) {
    return (4 * r0 + ((col >> 2) & 3u)) * 1024 + (col >> 4) * 64 + (col & 3u) * 16;
}

// Row index of v[k] before / after the column cores, and the first column of the tile.
template <int LOG_R>
__device__ __forceinline__ uint32_t col_row_strided(uint32_t r0, int k) { return r0 + ((uint32_t)k << (LOG_R - 4)); }
template <int LOG_R>
__device__ __forceinline__ uint32_t col_row_grouped(uint32_t r0, int k) { return 16 * r0 + (uint32_t)k; }

}  // namespace ks
