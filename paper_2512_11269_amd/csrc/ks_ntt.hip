// Negacyclic NTT / INTT for N = 2^12 .. 2^16 (Background, "NTT"; Kernel Code Generation, NTT kernels).
//
// A limb is viewed as an R x 256 matrix (row-major, R = N / 256).  The forward transform runs its first
// log2(R) decimation-in-time stages down the columns (butterfly partners R/2 ... 1 rows apart) and its last
// 8 stages inside the contiguous 256-point rows; the inverse mirrors it.  Each thread owns 16 points: four
// stages run in registers, then the tile is re-distributed through LDS for the next (up to) four.  Between the two kernels of
// a transform a limb is packed (ks_tiles.hpp); only the last kernel reduces to canonical residues.
#include <algorithm>

#include "ks_internal.hpp"
#include "ks_tasks.hpp"

namespace ks {

// Transforms of limbs of 64-bit words, in place.  Between the two passes a limb is packed inside its own bytes
// (in_place_offsets), 26 bytes moved per residue instead of 32; PACKED = false: doubles in the words' places (transform_packed).
__device__ __forceinline__ uint64_t* locate(const LimbMap& map, uint32_t li, uint64_t* data, uint64_t ps, uint32_t N, uint32_t* mod_id) {
    const uint32_t poly = li / map.n, idx = li - poly * map.n;
    *mod_id = map.mod[idx];
    return data + poly * ps + (uint64_t)map.off[idx] * N;
}

// forward, columns: canonical words in, packed lazy representatives out (|x| <= (1 + 0.501 log2 R) p).
template <int LOG_R, int TC, bool PACKED>
__global__ __launch_bounds__((TC << LOG_R) / 16) void ntt_fwd_cols(const double* __restrict__ tw, const Mod* __restrict__ mods, LimbMap map,
                                                        uint64_t* data, uint64_t ps) {
    constexpr uint32_t N = 256u << LOG_R, TILES = 256 / TC;
    __shared__ double lds[LOG_R > 4 ? (TC << LOG_R) : 1];
    const uint32_t tid = threadIdx.x, li = blockIdx.x / TILES, tile = blockIdx.x - li * TILES;
    uint32_t mod_id;
    uint64_t* limb = locate(map, li, data, ps, N, &mod_id);
    const Mod m = mods[mod_id];
    const uint32_t c = tid & (TC - 1), r0 = tid / TC, col = tile * TC + c;
    double v[16];
    PassTwiddles t;
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = u64_to_f64(limb[col_row_strided<LOG_R>(r0, k) * 256 + col]);
    load_col_twiddles<LOG_R>(t, tw + (size_t)mod_id * N, r0);
    col_fwd_core<LOG_R, TC>(v, t, c, r0, lds, m);
    if constexpr (PACKED) {
        tile_loaded<LOG_R>(v);
        in_place_store_cols<TC>(limb, r0, col, pack(v));
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) limb[col_row_grouped<LOG_R>(r0, k) * 256 + col] = __builtin_bit_cast(uint64_t, v[k]);
    }
}

// forward, rows: packed in, canonical words out.  One wavefront = four rows.  TC: columns of a tile of the column pass.
template <int LOG_R, int TC, bool PACKED>
__global__ __launch_bounds__(64) void ntt_fwd_rows(TwTables tw, const Mod* __restrict__ mods, LimbMap map, uint64_t* data, uint64_t ps) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R, GROUPS = R / 4;
    __shared__ double lds[4 * kRowPitch];
    const uint32_t lane = threadIdx.x, li = blockIdx.x / GROUPS, rg = blockIdx.x - li * GROUPS;
    uint32_t mod_id;
    uint64_t* limb = locate(map, li, data, ps, N, &mod_id);
    const Mod m = mods[mod_id];
    const uint32_t j0 = lane & 15, rr = lane >> 4, row = rg * 4 + rr;
    uint64_t* p = limb + row * 256 + j0;
    double v[16];
    PassTwiddles t;
    if constexpr (PACKED) {
        const PackedRaw raw = in_place_load_rows<TC>(limb, rg, lane);
        load_row_twiddles(t, tw, mod_id, N, R + row, j0, m);
        unpack_rows(raw, v);
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = __builtin_bit_cast(double, p[16 * k]);
        load_row_twiddles(t, tw, mod_id, N, R + row, j0, m);
    }
    row_fwd_core(v, t, j0, lds + rr * kRowPitch, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) p[16 * k] = f64_to_u64(canon(reduce_lazy(v[k], m), m));
}

// inverse, rows first: canonical words in, packed lazy representatives out (|x| <= 0.501 p).
template <int LOG_R, int TC, bool PACKED>
__global__ __launch_bounds__(64) void ntt_inv_rows(TwTables twi, const Mod* __restrict__ mods, LimbMap map, uint64_t* data, uint64_t ps) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R, GROUPS = R / 4;
    __shared__ double lds[4 * kRowPitch];
    const uint32_t lane = threadIdx.x, li = blockIdx.x / GROUPS, rg = blockIdx.x - li * GROUPS;
    uint32_t mod_id;
    uint64_t* limb = locate(map, li, data, ps, N, &mod_id);
    const Mod m = mods[mod_id];
    const uint32_t j0 = lane & 15, rr = lane >> 4, row = rg * 4 + rr;
    uint64_t* p = limb + row * 256 + j0;
    double v[16];
    PassTwiddles t;
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = u64_to_f64(p[16 * k]);
    load_row_twiddles(t, twi, mod_id, N, R + row, j0, m);
    row_inv_core(v, t, j0, lds + rr * kRowPitch, m);
    if constexpr (PACKED) {
        in_place_store_rows<TC>(limb, rg, lane, pack_rows(v));
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) p[16 * k] = __builtin_bit_cast(uint64_t, v[k]);
    }
}

// inverse, columns last: packed in; out = canonical [x N^-1]_m in words.
template <int LOG_R, int TC, bool PACKED>
__global__ __launch_bounds__((TC << LOG_R) / 16) void ntt_inv_cols(const double* __restrict__ twi, const Mod* __restrict__ mods,
                                                        const double* __restrict__ ninv, LimbMap map, uint64_t* data, uint64_t ps) {
    constexpr uint32_t N = 256u << LOG_R, TILES = 256 / TC;
    __shared__ double lds[LOG_R > 4 ? (TC << LOG_R) : 1];
    const uint32_t tid = threadIdx.x, li = blockIdx.x / TILES, tile = blockIdx.x - li * TILES;
    uint32_t mod_id;
    uint64_t* limb = locate(map, li, data, ps, N, &mod_id);
    const Mod m = mods[mod_id];
    const double scale = ninv[mod_id];
    const uint32_t c = tid & (TC - 1), r0 = tid / TC, col = tile * TC + c;
    double v[16];
    PassTwiddles t;
    if constexpr (PACKED) {
        const PackedRaw raw = in_place_load_cols<TC>(limb, r0, col);
        load_col_twiddles<LOG_R>(t, twi + (size_t)mod_id * N, r0);
        unpack(raw, v);
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = __builtin_bit_cast(double, limb[col_row_grouped<LOG_R>(r0, k) * 256 + col]);
        load_col_twiddles<LOG_R>(t, twi + (size_t)mod_id * N, r0);
    }
    col_inv_core<LOG_R, TC>(v, t, c, r0, lds, m);
    if constexpr (PACKED) tile_loaded<LOG_R>(v);
#pragma unroll
    for (int k = 0; k < 16; ++k) limb[col_row_strided<LOG_R>(r0, k) * 256 + col] = f64_to_u64(canon(mulmod_lazy(v[k], scale, m), m));
}

template <int W>
__device__ __forceinline__ void store_slot_words(uint32_t* p, const uint64_t* v) {
    struct alignas(W == 4 ? 16 : W == 2 ? 8 : 4) Words {
        uint32_t w[W];
    } o;
#pragma unroll
    for (int k = 0; k < W; ++k) o.w[k] = (uint32_t)v[k];
    *reinterpret_cast<Words*>(p) = o;
}

// The bundle the rotation gathers read (layout: GatherBundle), filled in one launch.  A workgroup owns four rows of one slab
// for all ciphertexts of the group, one wavefront per ciphertext: the first n_new workgroups run the row half of the
// forward transform on the raised limbs and leave canonical residues in LDS, from where every thread collects whole slots;
// the others copy the polynomial's own limbs into the slabs of their digits and the addend's limbs behind the digits.
// Interleaving here, once, makes the gathers of every rotation read 36 bytes per slot and digit for eight ciphertexts in runs
// of whole lines.
template <int LOG_R, int G, bool PACKED>
__global__ __launch_bounds__(64 * G) void gather_bundle_rows(TwTables tw, const Mod* __restrict__ mods, LimbMap map, DigitRanges dg,
                                                             uint32_t ell, uint32_t E, const uint8_t* __restrict__ lifted,
                                                             const void* __restrict__ d, const void* __restrict__ c0, uint64_t d_ps,
                                                             uint32_t n_new, uint32_t* __restrict__ lo, uint8_t* __restrict__ hi) {
    using WD = std::conditional_t<PACKED, uint64_t, uint32_t>;
    using Layout = SlotLayout<G>;
    using HW = typename Layout::HW;
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R, GROUPS = R / 4, TPB = 64 * G, WAVE_LDS = 4 * kRowPitch;
    constexpr uint32_t SLOTS = (1024 + TPB - 1) / TPB;  // slots of a thread; where G is no power of two the last one may be past the 1024
    __shared__ double lds[G * WAVE_LDS];
    const uint32_t tid = threadIdx.x;
    uint32_t slab, rg;
    uint64_t v[SLOTS * G];
    if (blockIdx.x < n_new) {  // uniform
        const uint32_t lane = tid & 63, j0 = lane & 15, rr = lane >> 4, w = tid >> 6;
        const uint32_t idx = blockIdx.x / GROUPS, mod_id = map.mod[idx];
        rg = blockIdx.x - idx * GROUPS;
        slab = map.off[idx];
        const Mod m = mods[mod_id];
        const uint32_t row = rg * 4 + rr;
        double x[16];
        PassTwiddles t;
        const PackedRaw raw = packed_load<64>(lifted + ((uint64_t)w * dg.ndig * E + slab) * packed_limb_bytes(N), N, rg * 256 + lane);
        load_row_twiddles(t, tw, mod_id, N, R + row, j0, m);
        unpack_rows(raw, x);
        double* lrow = lds + w * WAVE_LDS + rr * kRowPitch;
        row_fwd_core_consecutive(x, t, j0, lrow, m);
#pragma unroll
        for (int k = 0; k < 16; ++k) lrow[17 * j0 + k] = canon(reduce_lazy(x[k], m), m);
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < SLOTS; ++i) {
            const uint32_t s = tid + i * TPB, p = s & 255;
            if (s >= 1024) break;  // the same for a whole wavefront
#pragma unroll
            for (int g = 0; g < G; ++g) v[i * G + g] = f64_to_u64(lds[g * WAVE_LDS + (s >> 8) * kRowPitch + p + (p >> 4)]);
        }
    } else {
        const uint32_t t = blockIdx.x - n_new, li = t / GROUPS, pos = li < ell ? li : li - ell;
        rg = t - li * GROUPS;
        uint32_t j = 0;
        while (j + 1 < dg.ndig && pos >= dg.hi[j]) ++j;  // uniform
        slab = (li < ell ? j : dg.ndig) * E + pos;
        const WD* src = static_cast<const WD*>(li < ell ? d : c0) + (uint64_t)pos * N + rg * 1024 + tid;
#pragma unroll
        for (uint32_t i = 0; i < SLOTS; ++i) {
            if (tid + i * TPB >= 1024) break;
#pragma unroll
            for (uint32_t g = 0; g < G; ++g) v[i * G + g] = src[g * d_ps + i * TPB];
        }
    }
#pragma unroll
    for (uint32_t i = 0; i < SLOTS; ++i) {
        if (tid + i * TPB >= 1024) break;
        const uint64_t slot = (uint64_t)slab * N + rg * 1024 + tid + i * TPB;
        uint32_t h = 0;
        uint32_t* block = lo + (slot & ~63ull) * G;
        store_slot_words<Layout::FIRST>(block + (slot & 63) * Layout::FIRST, v + i * G);
        if constexpr (Layout::REST > 0) store_slot_words<Layout::REST>(block + 256 + (slot & 63) * Layout::REST, v + i * G + 4);
        if constexpr (PACKED) {
#pragma unroll
            for (int g = 0; g < G; ++g) h |= (uint32_t)(v[i * G + g] >> 32) << (4 * g);
            reinterpret_cast<HW*>(hi)[slot] = (HW)h;
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The inverse transform that feeds a conversion, packed limbs between its halves and at its end (ks_tiles.hpp).
// ------------------------------------------------------------------------------------------------
// W: 64- or 32-bit words of a tensor, or uint8_t: a packed limb of accumulators, then in place (in == out).
// in_ps: words (bytes for uint8_t) between polynomials, out_ps: bytes.
template <int LOG_R, typename W>
__global__ __launch_bounds__(64) void inv_rows_packed(TwTables twi, const Mod* __restrict__ mods, LimbMap map, const W* in, uint64_t in_ps,
                                                      uint8_t* out, uint64_t out_ps) {
    constexpr uint32_t N = 256u << LOG_R, GROUPS = (1u << LOG_R) / 4;
    __shared__ double lds[4 * kRowPitch];
    const uint32_t li = blockIdx.x / GROUPS, rg = blockIdx.x - li * GROUPS;
    const uint32_t poly = li / map.n, idx = li - poly * map.n, mod_id = map.mod[idx];
    const uint64_t limb = map.off[idx];
    task_inv_rows_packed<LOG_R, W>(twi, mods[mod_id], mod_id, in + poly * in_ps + limb * (sizeof(W) == 1 ? packed_limb_bytes(N) : N),
                                   out + poly * out_ps + limb * packed_limb_bytes(N), rg, threadIdx.x, lds);
}

// cta, ctb: [b][2][ell][N] words; dq: [b][2][ell], d2 and inv: [b][ell] packed limbs.
// Bound by its traffic, four limbs of words in and four packed ones out: eight pairs, 35 limbs, N = 2^16, 180 us (5.3 TB/s), where a
// tensor product by slots and the row half on its own took 166 + 50.
template <int LOG_R, typename W>
__global__ __launch_bounds__(64, 2) void tensor_inv_rows(TwTables twi, const Mod* __restrict__ mods, uint32_t ell, const W* __restrict__ cta,
                                                         const W* __restrict__ ctb, uint8_t* __restrict__ dq, uint8_t* __restrict__ d2,
                                                         uint8_t* __restrict__ inv) {
    constexpr uint32_t N = 256u << LOG_R;
    constexpr uint64_t LIMB = packed_limb_bytes(N);
    __shared__ double lds[4 * kRowPitch];
    const uint32_t rg = blockIdx.x, i = blockIdx.y, b = blockIdx.z;
    const uint64_t ct = ((uint64_t)b * 2 * ell + i) * N, one = (uint64_t)b * ell + i, two = (uint64_t)b * 2 * ell + i;
    task_tensor_inv_rows<LOG_R, W>(twi, mods[i], i, cta + ct, ctb + ct, (uint64_t)ell * N, dq + two * LIMB, dq + (two + ell) * LIMB, d2 + one * LIMB,
                                   inv + one * LIMB, rg, threadIdx.x, lds);
}

// Out: [x * scale]_m as sources of a conversion; scale_tab holds N^-1 times the conversion's (D / s_i)^-1, by position in the map.
template <int LOG_R>
__global__ __launch_bounds__(256) void inv_cols_packed(const double* __restrict__ twi, const Mod* __restrict__ mods,
                                                       const double* __restrict__ scale_tab, LimbMap map, uint8_t* data, uint64_t ps) {
    constexpr uint32_t N = 256u << LOG_R, TILES = 1u << (LOG_R - 4);
    __shared__ double lds[LOG_R > 4 ? 4096 : 1];
    const uint32_t li = blockIdx.x / TILES, tile = blockIdx.x - li * TILES;
    const uint32_t poly = li / map.n, idx = li - poly * map.n, mod_id = map.mod[idx];
    task_inv_cols_packed<LOG_R>(twi + (size_t)mod_id * N, mods[mod_id], scale_tab[idx],
                                data + poly * ps + (uint64_t)map.off[idx] * packed_limb_bytes(N), tile, threadIdx.x, lds);
}

// ------------------------------------------------------------------------------------------------
// Transforms of limbs held in 32-bit words (every modulus below 2^32), in place.  Both passes read and write canonical
// residues, so the half-way values fit the same words and a transform moves half the bytes of the 64-bit one.
// fwd_cols -> fwd_rows, inv_rows -> inv_cols as above.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t* locate_u32(const LimbMap& map, uint32_t li, uint32_t* data, uint64_t ps, uint32_t N,
                                                uint32_t* mod_id) {
    const uint32_t poly = li / map.n, idx = li - poly * map.n;
    *mod_id = map.mod[idx];
    return data + poly * ps + (uint64_t)map.off[idx] * N;
}

template <int LOG_R, int TC>
__global__ __launch_bounds__((TC << LOG_R) / 16) void ntt_fwd_cols_u32(const double* __restrict__ tw, const Mod* __restrict__ mods,
                                                                     LimbMap map, uint32_t* data, uint64_t ps) {
    constexpr uint32_t N = 256u << LOG_R, TILES = 256 / TC;
    __shared__ double lds[LOG_R > 4 ? (TC << LOG_R) : 1];
    const uint32_t tid = threadIdx.x, li = blockIdx.x / TILES, tile = blockIdx.x - li * TILES;
    uint32_t mod_id;
    uint32_t* p = locate_u32(map, li, data, ps, N, &mod_id);
    const Mod m = mods[mod_id];
    const uint32_t c = tid & (TC - 1), r0 = tid / TC, col = tile * TC + c;
    double v[16];
    PassTwiddles t;
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = (double)p[col_row_strided<LOG_R>(r0, k) * 256 + col];
    load_col_twiddles<LOG_R>(t, tw + (size_t)mod_id * N, r0);
    col_fwd_core<LOG_R, TC>(v, t, c, r0, lds, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) p[col_row_grouped<LOG_R>(r0, k) * 256 + col] = (uint32_t)canon(reduce_lazy(v[k], m), m);
}

template <int LOG_R, bool INVERSE>
__global__ __launch_bounds__(64) void ntt_rows_u32(TwTables tw, const Mod* __restrict__ mods, LimbMap map, uint32_t* data,
                                                   uint64_t ps) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R, GROUPS = R / 4;
    __shared__ double lds[4 * kRowPitch];
    const uint32_t tid = threadIdx.x, li = blockIdx.x / GROUPS, rg = blockIdx.x - li * GROUPS;
    uint32_t mod_id;
    uint32_t* limb = locate_u32(map, li, data, ps, N, &mod_id);
    const Mod m = mods[mod_id];
    const uint32_t j0 = tid & 15, rr = tid >> 4, row = rg * 4 + rr;
    uint32_t* p = limb + row * 256;
    double v[16];
    PassTwiddles t;
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = (double)p[j0 + 16 * k];
    load_row_twiddles(t, tw, mod_id, N, R + row, j0, m);
    if constexpr (INVERSE) row_inv_core(v, t, j0, lds + rr * kRowPitch, m);
    else row_fwd_core(v, t, j0, lds + rr * kRowPitch, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) p[j0 + 16 * k] = (uint32_t)canon(reduce_lazy(v[k], m), m);
}

template <int LOG_R, int TC>
__global__ __launch_bounds__((TC << LOG_R) / 16) void ntt_inv_cols_u32(const double* __restrict__ twi, const Mod* __restrict__ mods,
                                                                     const double* __restrict__ ninv, LimbMap map, uint32_t* data,
                                                                     uint64_t ps) {
    constexpr uint32_t N = 256u << LOG_R, TILES = 256 / TC;
    __shared__ double lds[LOG_R > 4 ? (TC << LOG_R) : 1];
    const uint32_t tid = threadIdx.x, li = blockIdx.x / TILES, tile = blockIdx.x - li * TILES;
    uint32_t mod_id;
    uint32_t* p = locate_u32(map, li, data, ps, N, &mod_id);
    const Mod m = mods[mod_id];
    const double scale = ninv[mod_id];
    const uint32_t c = tid & (TC - 1), r0 = tid / TC, col = tile * TC + c;
    double v[16];
    PassTwiddles t;
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = (double)p[col_row_grouped<LOG_R>(r0, k) * 256 + col];
    load_col_twiddles<LOG_R>(t, twi + (size_t)mod_id * N, r0);
    col_inv_core<LOG_R, TC>(v, t, c, r0, lds, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) p[col_row_strided<LOG_R>(r0, k) * 256 + col] = (uint32_t)canon(mulmod_lazy(v[k], scale, m), m);
}

// ------------------------------------------------------------------------------------------------
// Wide tiles (32 columns, 256-byte segments) move more bytes per second but give half as many workgroups;
// small launches keep the 16-column tiles.
static bool wide_tiles(uint32_t limbs) { return limbs >= 256; }

void launch_gather_bundle_rows(const ks_ctx* c, const Level& lv, const uint8_t* lifted, const void* d, const void* c0, uint64_t ps_words,
                               const GatherBundle& out, bool raised, hipStream_t s) {
    const uint32_t n_new = raised ? lv.lifted_map.n : 0, n_copy = c0 ? 2 * lv.ell : lv.ell;
    DigitRanges dg;
    dg.ndig = lv.ndig;
    for (uint32_t j = 0; j < kMaxDigits; ++j) {
        dg.lo[j] = j < lv.ndig ? lv.digit_lo[j] : 0;
        dg.hi[j] = j < lv.ndig ? lv.digit_hi[j] : 0;
    }
    const double wb = 4.0 + (out.hi ? (double)gather_hi_bytes(out.group) / out.group : 0.0);
    ProfScope ps("gather_bundle_rows", ((5.0 + wb) * n_new + ((out.hi ? 8.0 : 4.0) + wb) * n_copy) * c->N * out.group, s);
    const uint32_t groups = c->N / 1024;
#define KS_LAUNCH_BUNDLE(LOGR, GV, PK)                                                                                               \
    hipLaunchKernelGGL((gather_bundle_rows<LOGR, GV, PK>), dim3((n_new + n_copy) * groups), dim3(64 * GV), 0, s, c->tw_fwd, c->d_mod,  \
                       lv.lifted_map, dg, lv.ell, lv.E, lifted, d, c0, ps_words, n_new * groups, out.lo, out.hi)
#define KS_LAUNCH(LOGR)                                              \
    {                                                                \
        constexpr int kLogR = LOGR;                                  \
        if (out.hi) { KS_FOR_GROUP(out.group, KS_LAUNCH_PACKED) }    \
        else { KS_FOR_GROUP(out.group, KS_LAUNCH_WORDS32) }          \
    }
#define KS_LAUNCH_PACKED(GV) KS_LAUNCH_BUNDLE(kLogR, GV, true)
#define KS_LAUNCH_WORDS32(GV) KS_LAUNCH_BUNDLE(kLogR, GV, false)
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_PACKED
#undef KS_LAUNCH_WORDS32
#undef KS_LAUNCH_BUNDLE
}

// Polynomials per launch pair of a two-pass transform: the second pass of a group should find what the first pass wrote
// still in the 256 MB last-level cache.  Measured on 1920 limbs: groups of 240 MB are 8 % faster than one pair of launches
// over everything, groups of 64 MB 9 % slower (launches too small), groups of 320 MB no different.
static uint32_t polys_per_group(const ks_ctx* c, const LimbMap& map) {
    constexpr uint64_t kGroupBytes = 240ull << 20;
    const uint64_t poly_bytes = (uint64_t)map.n * c->N * 8;
    return (uint32_t)std::max<uint64_t>(1, kGroupBytes / poly_bytes);
}

// Whether a launch of the 64-bit transforms packs its limbs between the two passes.  Not at N <= 2^14 for data of about what the eight
// L2s hold together (32 MB): the second pass, which writes whole limbs and then has read five eighths of their lines, takes 2 to 4.5 us
// longer there, more than the first one gains.  Calls as doubles / packed, us, by MiB of data (elsewhere packed is up to 18 % ahead):
//   inverse, N = 2^12: 18 25.2 / 24.7, 21 24.5 / 26.1, 23 23.6 / 25.9, 27 24.3 / 24.9, 32 24.6 / 24.4; N = 2^13: 17 31.5 / 30.1, 21 25.6 / 30.7,
// 24 22.7 / 26.2, 32 24.6 / 28.1, 36 28.8 / 28.5; N = 2^14: 18 28.4 / 27.6, 19 27.7 / 28.0, 27 25.8 / 27.9, 35 28.1 / 28.6, 36 28.6 / 28.5
//   forward, N = 2^12: 20 24.9 / 24.8, 23 23.5 / 25.2, 26 24.2 / 24.6, 28 24.9 / 23.8; N = 2^13: 18 25.2 / 24.7, 21 22.5 / 25.4, 25 24.0 / 24.7, 26 25.4 / 23.5;
// N = 2^14: 18 27.1 / 26.9, 22 24.9 / 26.8, 32 24.7 / 25.4, 34 28.0 / 27.6
//   Just past these lines GPUs differ by 4 % either way, as they do at N = 2^15; at 2^16 the packed form is between 2 % behind and 11 % ahead.
static bool transform_packed(const ks_ctx* c, uint32_t limbs, bool inverse) {
    if (c->logN > 14) return true;
    const uint64_t bytes = 8ull * limbs * c->N, mib = 1 << 20;
    const uint64_t most = inverse ? (c->logN == 12 ? 28 : 35) : (c->logN == 12 ? 26 : c->logN == 13 ? 25 : 33);
    return bytes < 19 * mib || bytes > most * mib;
}

void launch_ntt(const ks_ctx* c, const LimbMap& map, uint64_t* data, uint64_t ps_words, uint32_t n_polys, bool inverse, hipStream_t s) {
    const uint32_t g = polys_per_group(c, map);
    for (uint32_t p0 = 0; p0 < n_polys; p0 += g) {
        const uint32_t limbs = map.n * std::min(g, n_polys - p0);
        uint64_t* part = data + (uint64_t)p0 * ps_words;
        const bool packed = transform_packed(c, limbs, inverse);
        const double bytes = (packed ? 13.0 : 16.0) * limbs * c->N;
#define KS_LAUNCH_TC(LOGR, TCV, PK)                                                                                                       \
    {                                                                                                                                     \
        const dim3 cols(limbs * (256 / TCV)), cols_block((TCV << LOGR) / 16), rows(limbs << (LOGR - 2)), rows_block(64);                  \
        if (!inverse) {                                                                                                                   \
            {                                                                                                                             \
                ProfScope ps("ntt_fwd_cols", bytes, s);                                                                                   \
                hipLaunchKernelGGL((ntt_fwd_cols<LOGR, TCV, PK>), cols, cols_block, 0, s, c->d_tw_fwd, c->d_mod, map, part, ps_words);    \
            }                                                                                                                             \
            ProfScope ps("ntt_fwd_rows", bytes, s);                                                                                       \
            hipLaunchKernelGGL((ntt_fwd_rows<LOGR, TCV, PK>), rows, rows_block, 0, s, c->tw_fwd, c->d_mod, map, part, ps_words);          \
        } else {                                                                                                                          \
            {                                                                                                                             \
                ProfScope ps("ntt_inv_rows", bytes, s);                                                                                   \
                hipLaunchKernelGGL((ntt_inv_rows<LOGR, TCV, PK>), rows, rows_block, 0, s, c->tw_inv, c->d_mod, map, part, ps_words);      \
            }                                                                                                                             \
            ProfScope ps("ntt_inv_cols", bytes, s);                                                                                       \
            hipLaunchKernelGGL((ntt_inv_cols<LOGR, TCV, PK>), cols, cols_block, 0, s, c->d_tw_inv, c->d_mod, c->d_ninv, map, part, ps_words); \
        }                                                                                                                                 \
    }
#define KS_LAUNCH(LOGR)                                                     \
    if constexpr (LOGR > 6) KS_LAUNCH_TC(LOGR, (4096 >> LOGR), true)        \
    else if (packed) KS_LAUNCH_TC(LOGR, (4096 >> LOGR), true)               \
    else KS_LAUNCH_TC(LOGR, (4096 >> LOGR), false)
        if (c->logN == 16 && wide_tiles(limbs)) KS_LAUNCH_TC(8, 32, true)
        else KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_TC
    }
}

void launch_inv_rows_packed(const ks_ctx* c, const LimbMap& map, const void* in, uint64_t in_ps, int in_word, uint8_t* out, uint64_t out_ps,
                            uint32_t n_polys, hipStream_t s) {
    const uint32_t limbs = map.n * n_polys;
    if (limbs == 0) return;
    ProfScope ps("inv_rows_packed", ((in_word == 1 ? 5.0 : in_word) + 5.0) * limbs * c->N, s);
#define KS_LAUNCH_W(LOGR, WT)                                                                                                          \
    hipLaunchKernelGGL((inv_rows_packed<LOGR, WT>), dim3(limbs << (LOGR - 2)), dim3(64), 0, s, c->tw_inv, c->d_mod, map,               \
                       static_cast<const WT*>(in), in_ps, out, out_ps)
#define KS_LAUNCH(LOGR)                               \
    if (in_word == 1) KS_LAUNCH_W(LOGR, uint8_t);     \
    else if (in_word == 4) KS_LAUNCH_W(LOGR, uint32_t); \
    else KS_LAUNCH_W(LOGR, uint64_t)
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_W
}

void launch_tensor_inv_rows(const ks_ctx* c, const void* cta, const void* ctb, uint32_t ell, uint8_t* dq, uint8_t* d2, uint8_t* inv,
                            uint32_t batch, hipStream_t s, bool in_words32) {
    if (batch == 0) return;
    ProfScope ps("tensor_inv_rows", (double)batch * ell * ((in_words32 ? 16 : 32) + 20) * c->N, s);
#define KS_LAUNCH_W(LOGR, WT)                                                                                                    \
    hipLaunchKernelGGL((tensor_inv_rows<LOGR, WT>), dim3(c->N / 1024, ell, batch), dim3(64), 0, s, c->tw_inv, c->d_mod, ell,     \
                       static_cast<const WT*>(cta), static_cast<const WT*>(ctb), dq, d2, inv)
#define KS_LAUNCH(LOGR)                        \
    if (in_words32) KS_LAUNCH_W(LOGR, uint32_t); \
    else KS_LAUNCH_W(LOGR, uint64_t)
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_W
}

void launch_inv_cols_packed(const ks_ctx* c, const LimbMap& map, uint8_t* data, uint64_t ps_bytes, uint32_t n_polys, const double* scale_tab,
                            hipStream_t s) {
    const uint32_t limbs = map.n * n_polys;
    if (limbs == 0) return;
    ProfScope ps("inv_cols_packed", 2.0 * limbs * packed_limb_bytes(c->N), s);
#define KS_LAUNCH(LOGR)                                                                                                              \
    hipLaunchKernelGGL((inv_cols_packed<LOGR>), dim3(limbs << (LOGR - 4)), dim3(256), 0, s, c->d_tw_inv, c->d_mod, scale_tab, map, data, \
                       ps_bytes)
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
}

void launch_ntt_u32(const ks_ctx* c, const LimbMap& map, uint32_t* data, uint64_t ps_words, uint32_t n_polys, bool inverse,
                    hipStream_t s) {
    // groups sized like the 64-bit transform's: the second pass should find the first pass's output in the last-level cache
    const uint32_t g = 2 * polys_per_group(c, map);
    for (uint32_t p0 = 0; p0 < n_polys; p0 += g) {
        const uint32_t limbs = map.n * std::min(g, n_polys - p0);
        uint32_t* part = data + (uint64_t)p0 * ps_words;
        // column tiles: 32 columns at N = 2^16 (128-byte row segments of 32-bit words), 4096 / R otherwise
#define KS_LAUNCH_TC(LOGR, TCV)                                                                                                     \
    if (!inverse) {                                                                                                                 \
        {                                                                                                                           \
            ProfScope ps("ntt_fwd_cols_u32", 1.0 * limbs * c->N * 8.0, s);                                                          \
            hipLaunchKernelGGL((ntt_fwd_cols_u32<LOGR, TCV>), dim3(limbs * (256 / TCV)), dim3((TCV << LOGR) / 16), 0, s,            \
                               c->d_tw_fwd, c->d_mod, map, part, ps_words);                                                        \
        }                                                                                                                           \
        ProfScope ps("ntt_fwd_rows_u32", 1.0 * limbs * c->N * 8.0, s);                                                              \
        hipLaunchKernelGGL((ntt_rows_u32<LOGR, false>), dim3(limbs << (LOGR - 2)), dim3(64), 0, s, c->tw_fwd, c->d_mod, map, part,  \
                           ps_words);                                                                                              \
    } else {                                                                                                                        \
        {                                                                                                                           \
            ProfScope ps("ntt_inv_rows_u32", 1.0 * limbs * c->N * 8.0, s);                                                          \
            hipLaunchKernelGGL((ntt_rows_u32<LOGR, true>), dim3(limbs << (LOGR - 2)), dim3(64), 0, s, c->tw_inv, c->d_mod, map,     \
                               part, ps_words);                                                                                    \
        }                                                                                                                           \
        ProfScope ps("ntt_inv_cols_u32", 1.0 * limbs * c->N * 8.0, s);                                                              \
        hipLaunchKernelGGL((ntt_inv_cols_u32<LOGR, TCV>), dim3(limbs * (256 / TCV)), dim3((TCV << LOGR) / 16), 0, s, c->d_tw_inv,   \
                           c->d_mod, c->d_ninv, map, part, ps_words);                                                              \
    }
        switch (c->logN) {
            case 12: KS_LAUNCH_TC(4, 256) break;
            case 13: KS_LAUNCH_TC(5, 128) break;
            case 14: KS_LAUNCH_TC(6, 64) break;
            case 15: KS_LAUNCH_TC(7, 32) break;
            default: KS_LAUNCH_TC(8, 32) break;
        }
#undef KS_LAUNCH_TC
    }
}

}  // namespace ks
