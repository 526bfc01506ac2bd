// The bodies of the pipeline kernels as device functions over explicit tile coordinates (the kernels in ks_ntt.hip,
// ks_fused.hip and ks_bconv_mfma.hip map their block indices onto them).  "Wave tasks" are executed by one wavefront (lane = threadIdx.x % 64) on four 256-point rows and need
// 4 * kRowPitch doubles of LDS of their own; "workgroup tasks" are executed by 256 threads on a column tile.
// Every task contains the same number of workgroup barriers for all its threads.
#pragma once
#include "ks_internal.hpp"
#include "ks_tiles.hpp"

namespace ks {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// ---- inverse transform, row half, for a conversion: canonical residues (W words) or a packed limb of accumulators (uint8_t) in,
// a packed limb in columns order out (in place where the input is packed).
template <int LOG_R, typename W>
__device__ __forceinline__ void task_inv_rows_packed(const TwTables& twi, Mod m, uint32_t mod_id, const W* ip, uint8_t* op, uint32_t rg,
                                                     uint32_t lane, double* lds_wave) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R;
    const uint32_t j0 = lane & 15, rr = lane >> 4, row = rg * 4 + rr;
    double v[16];
    PassTwiddles t;
    if constexpr (sizeof(W) == 1) {
        const PackedRaw raw = packed_load<64>(ip, N, rg * 256 + lane);
        unpack(raw, v);
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = word_to_f64<W>(ip[row * 256 + j0 + 16 * k]);
    }
    load_row_twiddles(t, twi, mod_id, N, R + row, j0, m);
    row_inv_core(v, t, j0, lds_wave + rr * kRowPitch, m);
    packed_store<64>(op, N, rg * 256 + lane, pack_rows(v));
}

// ---- tensor product of two ciphertexts (b1, a1) x (b2, a2) and the row half of the inverse transform of a1 a2 -----------
// One wavefront: four rows (group rg) of one limb.  d0 = b1 b2 and d1 = a1 b2 + a2 b1 are only added back by the last kernel of the
// call, d2 = a1 a2 is one digit of the inner product as it is: packed, rows order.  inv: the transformed d2, columns order.
// x1 / x2: that limb of b1 and b2, the limbs of a1 and a2 `comp` words behind.
template <int LOG_R, typename W>
__device__ __forceinline__ void task_tensor_inv_rows(const TwTables& twi, Mod m, uint32_t mod_id, const W* __restrict__ x1,
                                                     const W* __restrict__ x2, uint64_t comp, uint8_t* __restrict__ d0, uint8_t* __restrict__ d1,
                                                     uint8_t* __restrict__ d2, uint8_t* __restrict__ inv, uint32_t rg, uint32_t lane,
                                                     double* lds_wave) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R;
    const uint32_t j0 = lane & 15, rr = lane >> 4, row = rg * 4 + rr, off = row * 256 + j0, at = rg * 256 + lane;
    W b1[16], a1[16], b2[16], a2[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        a1[k] = x1[comp + off + 16 * k];
        a2[k] = x2[comp + off + 16 * k];
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        b1[k] = x1[off + 16 * k];
        b2[k] = x2[off + 16 * k];
    }
    PassTwiddles t;
    double v[16], u[16];
#pragma unroll
    for (int k = 0; k < 16; ++k)
        u[k] = reduce_lazy(mulmod_lazy(word_to_f64<W>(a1[k]), word_to_f64<W>(b2[k]), m) + mulmod_lazy(word_to_f64<W>(a2[k]), word_to_f64<W>(b1[k]), m), m);
    packed_store<64>(d1, N, at, pack(u));
#pragma unroll
    for (int k = 0; k < 16; ++k) u[k] = mulmod_lazy(word_to_f64<W>(b1[k]), word_to_f64<W>(b2[k]), m);
    packed_store<64>(d0, N, at, pack(u));
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = mulmod_lazy(word_to_f64<W>(a1[k]), word_to_f64<W>(a2[k]), m);
    packed_store<64>(d2, N, at, pack(v));
    load_row_twiddles(t, twi, mod_id, N, R + row, j0, m);
    row_inv_core(v, t, j0, lds_wave + rr * kRowPitch, m);
    packed_store<64>(inv, N, at, pack_rows(v));
}

// ---- inverse transform, column half, for a conversion: a packed limb in columns order in, the sources of the conversion out, in place ----------
template <int LOG_R>
__device__ __forceinline__ void task_inv_cols_packed(const double* __restrict__ Wi, Mod m, double scale, uint8_t* limb, uint32_t tile,
                                                     uint32_t tid, double* lds) {
    constexpr uint32_t N = 256u << LOG_R, TC = 4096u >> LOG_R;
    const uint32_t c = tid & (TC - 1), r0 = tid / TC, col = tile * TC + c, at = r0 * 1024 + col;
    double v[16];
    PassTwiddles t;
    const PackedRaw raw = packed_load<256>(limb, N, at);
    load_col_twiddles<LOG_R>(t, Wi, r0);
    unpack(raw, v);
    col_inv_core<LOG_R, TC>(v, t, c, r0, lds, m);
    tile_loaded<LOG_R>(v);
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = canon(mulmod_lazy(v[k], scale, m), m);
    const PackedRaw o = pack(v, kDigitBias);
    Words4* lo = reinterpret_cast<Words4*>(limb) + at;
#pragma unroll
    for (int q = 0; q < 4; ++q) lo[q * 256] = Words4{{o.lo[4 * q], o.lo[4 * q + 1], o.lo[4 * q + 2], o.lo[4 * q + 3]}};
    *reinterpret_cast<Words4*>(limb + 4 * N + source_bytes_offset(r0, col)) = Words4{{o.hi[0], o.hi[1], o.hi[2], o.hi[3]}};
}

// ---- base conversion on the matrix cores + column half of the forward transform (see ks_bconv_mfma.hip) --------------
// Twiddles of the column butterflies, staged in LDS (both lane halves of a workgroup need different tables, so they
// cannot ride in scalar registers, and 30 vector registers per target would cost a wavefront of occupancy):
//   first pass : entries 1..15 = W[j], the sub-tree below heap node 1, the same for every thread of a half;
//   second pass: for every row group r0, entries (1 << ul) + g = W[(1 << (E + ul)) + (r0 << ul) + g] for the last E local
//                stages ul = 4 - E .. 3 (for E = 4 the sub-tree below node 16 + r0).
// Layout per (half, target): [1 + S][16] doubles, S = R / 16 row groups.
template <int LOG_R>
__device__ __forceinline__ uint32_t col_twiddle_index(uint32_t slot, uint32_t j) {
    constexpr int E = LOG_R - 4;
    if (j == 0) return 0;
    if (slot == 0) return j;
    const uint32_t ul = 31u - __clz(j), g = j - (1u << ul), r0 = slot - 1;
    return (int)ul >= 4 - E ? (1u << (E + ul)) + (r0 << ul) + g : 0u;
}

template <int LOG_R, int TL, int WAVES>
struct MfmaConvShape {
    static constexpr uint32_t R = 1u << LOG_R, TC = (512u * WAVES) >> LOG_R;  // tile: TC columns x R rows, 512 positions a wavefront
    static constexpr int E = LOG_R - 4, S = 1 << E;
    // exchange buffer of the column butterflies, one region per lane half; rows are padded so that the 16-row groups the
    // second pass reads start in different banks
    static constexpr uint32_t PADW = TC <= 16 ? TC : 0, HALF_WORDS = R * TC + (R / 16) * PADW;
    static constexpr uint32_t TW_WORDS = (1 + S) * 16;  // per (half, target)
    static constexpr uint32_t LDS_WORDS = LOG_R > 4 ? 2 * HALF_WORDS : 1, LDS_TW_WORDS = 2 * TL * TW_WORDS;
};

// 64 WAVES threads; y / out: the source and output bundles (y_ps and out_ps bytes a polynomial) of polynomials poly0, + step, ... below
// n_polys; tile: 512 WAVES positions; t0: first of the 2 TL targets (t0 < n_dst); lds: LDS_WORDS doubles; lds_tw: LDS_TW_WORDS doubles.
// The sources of the next polynomial are requested after the first target of the current one, into the registers that its
// conversion and that target have freed; factors and twiddles are fetched once.
template <int LOG_R, int TL, int T, int WAVES>
__device__ __forceinline__ void task_bconv_mfma_cols(const double* __restrict__ tw, const BConvPlan& P, const PlanMeta& PM,
                                                     const uint8_t* __restrict__ y, uint64_t y_ps, uint8_t* __restrict__ out, uint64_t out_ps,
                                                     uint32_t poly0, uint32_t step, uint32_t n_polys, uint32_t tile, int t0, uint32_t tid,
                                                     double* lds, double* lds_tw) {
    using Shape = MfmaConvShape<LOG_R, TL, WAVES>;
    constexpr int NM = mfma_instructions(T);
    constexpr uint32_t N = 256u << LOG_R, TC = Shape::TC, PADW = Shape::PADW, HALF_WORDS = Shape::HALF_WORDS, TW_WORDS = Shape::TW_WORDS;
    constexpr int E = Shape::E, S = Shape::S;
    const uint32_t lane = tid & 63u, h = lane >> 5, p = (tid >> 6) * 32u + (lane & 31u);
    const uint32_t c = p & (TC - 1), r0 = p / TC, col = tile * TC + c;
    const int n_dst = (int)PM.n_dst;

    // B operand: the sources of this lane's slots, already cut into digits (kDigitBias), read through a buffer descriptor
    // (per-lane offset = position + limb).  A source of the 16 positions is four accesses of 16 bytes and, for the fifth
    // digits, one more.  The first ones are requested before anything else.
    uint32_t voff[T];
    // quads of positions whose loads are in flight together, and whether position k - 1 is recombined under the matrix
    // instructions of position k (a second set of result registers) or right away: the single-target shape is kept within 128 registers
    constexpr int QB = TL == 1 ? (T <= 2 ? 2 : 1) : T <= 2 ? 4 : T <= 4 ? 3 : 1;
    constexpr bool OVERLAP = TL > 1 && T <= 4;
    const uint32_t top_off = source_bytes_offset(r0, col) + 4 * N - (r0 * 1024 + col) * 16;   // from a source's first quad
    Words4 yq[QB][T], ytop[T];
    BufferRsrc ysrd;
    const auto load4 = [&](uint32_t lane_off, uint32_t off) {
        return __builtin_bit_cast(Words4, __builtin_amdgcn_raw_buffer_load_b128(ysrd, (int)lane_off, (int)off, 0));
    };
    const auto request = [&](uint32_t poly) {
        ysrd = make_buffer_rsrc(y + (uint64_t)poly * y_ps, y_ps);
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
            for (int e = 0; e < T; ++e) {
                yq[q][e] = load4(voff[e], q * 4096);
                if (q == 0) ytop[e] = load4(voff[e] + top_off, 0);
            }
    };
#pragma unroll
    for (int e = 0; e < T; ++e) {
        // both candidates through scalar registers (a select between two loads would become one per-lane load)
        const int at = 6 * mfma_slot_of(T, e) + e - mfma_slot_start(T, mfma_slot_of(T, e));
        const uint32_t limb0 = __builtin_amdgcn_readfirstlane(PM.src_limb[at]), limb1 = __builtin_amdgcn_readfirstlane(PM.src_limb[at + 3]);
        voff[e] = (h ? limb1 : limb0) * (uint32_t)packed_limb_bytes(N) + (r0 * 1024 + col) * 16;
    }
    request(poly0);

    // A operand: this lane's row of the factor matrix.  Result register j = 5 u + b sits in row 8 (j / 4) + 4 h' + j % 4,
    // so row r belongs to lane half h' = (r / 4) % 2 and register j = 4 (r / 8) + r % 4.
    v4i afac[NM];
    {
        const uint32_t r = lane & 31u, hp = (r >> 2) & 1u, j = 4 * (r >> 3) + (r & 3u), u = j / 5, b = j - 5 * u;
        const int ta = min(t0 + (int)(hp * TL + u), n_dst - 1);  // a ragged last subset recomputes the last target
        const bool used = u < (uint32_t)TL;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const v4i* row = reinterpret_cast<const v4i*>(&P.afac[ta][b][2 * m + h][0]);
            afac[m] = used ? *row : v4i{0, 0, 0, 0};
        }
    }
    // per-lane constants of the targets this lane half receives: one 32-byte record each
    Mod mt[TL];
    int tgt[TL];
    uint32_t dst_limb[TL];
#pragma unroll
    for (int u = 0; u < TL; ++u) {
        tgt[u] = t0 + (int)h * TL + u;
        const BConvPlan::TargetRec rec = P.trec[min(tgt[u], n_dst - 1)];
        mt[u] = rec.m;
        dst_limb[u] = rec.limb;
    }
    // twiddles of all 2 TL targets -> LDS (used after a barrier)
    constexpr uint32_t THREADS = 64 * WAVES;
    constexpr int TW_PER_THREAD = (2 * TL * TW_WORDS + THREADS - 1) / THREADS;
    double twv[TW_PER_THREAD];
#pragma unroll
    for (int i = 0; i < TW_PER_THREAD; ++i) {
        const uint32_t w = min(tid + THREADS * i, 2u * TL * TW_WORDS - 1), ht = w / TW_WORDS, rem = w - ht * TW_WORDS;
        const int t = min(t0 + (int)ht, n_dst - 1);  // ht = half * TL + u, the order of the targets
        twv[i] = tw[(size_t)P.trec[t].mod_id * N + col_twiddle_index<LOG_R>(rem >> 4, rem & 15u)];
    }

#pragma unroll
    for (int i = 0; i < TW_PER_THREAD; ++i)
        if (tid + THREADS * i < 2u * TL * TW_WORDS) lds_tw[tid + THREADS * i] = twv[i];

    // Software pipeline over the 16 positions, fenced per position so that the schedule below is the one that runs
    // (left alone, the scheduler hoists every matrix instruction and spills): issue the matrix instructions of position k,
    // re-request the registers of a quad of positions when its last one is done, then recombine position k - 1, whose
    // results have had a whole position's worth of instructions to arrive.
    double acc[TL][16];
    v16i sums[OVERLAP ? 2 : 1];
    auto recombine = [&](int k) {
        const v16i& s = sums[OVERLAP ? (k & 1) : 0];
#pragma unroll
        for (int u = 0; u < TL; ++u) {
            // sum_b 256^b S_b: the two low pairs fit 32-bit integers, the rest is exact in doubles
            const int lo = s[5 * u] + (s[5 * u + 1] << 8), mid = s[5 * u + 2] + (s[5 * u + 3] << 8);
            const double v = __builtin_fma((double)s[5 * u + 4], 4294967296.0, __builtin_fma((double)mid, 65536.0, (double)lo));
            acc[u][k] = reduce_lazy(v, mt[u]);
            // pin the recombined value here: otherwise the optimiser sinks these few instructions down to the butterflies
            // and keeps the 16 raw sums of every position alive instead (spilling them)
            asm volatile("" : "+v"(acc[u][k]));
        }
    };
#pragma unroll 1
    for (uint32_t poly = poly0; poly < n_polys; poly += step) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int q = k / 4, x = k % 4;
            v16i s = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                constexpr int LAST = T - 1;
                const int e0 = mfma_slot_start(T, m), n = mfma_slot_sources(T, m);
                v4i bq = {(int)(yq[q % QB][e0].w[x] ^ 0x80808080u), 0, 0, 0};
                if (n > 1) bq[1] = (int)(yq[q % QB][min(e0 + 1, LAST)].w[x] ^ 0x80808080u);
                if (n > 2) bq[2] = (int)(yq[q % QB][min(e0 + 2, LAST)].w[x] ^ 0x80808080u);
                // byte x of the sources' fifth digits
                uint32_t top = __builtin_amdgcn_perm(n > 1 ? ytop[min(e0 + 1, LAST)].w[q] : 0u, ytop[e0].w[q], 0x0c0c0000u + (n > 1 ? (x + 4) << 8 : 0xc00) + x);
                if (n > 2) top = __builtin_amdgcn_perm(ytop[min(e0 + 2, LAST)].w[q], top, 0x0c000100u + ((x + 4) << 16));
                bq[3] = (int)top;
                s = __builtin_amdgcn_mfma_i32_32x32x32_i8(afac[m], bq, s, 0, 0, 0);
            }
            if (x == 3 && q + QB < 4) {
#pragma unroll
                for (int e = 0; e < T; ++e) yq[q % QB][e] = load4(voff[e], (q + QB) * 4096);
            }
            sums[OVERLAP ? (k & 1) : 0] = s;
            if (!OVERLAP) recombine(k);
            else if (k > 0) recombine(k - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (OVERLAP) recombine(15);
        __syncthreads();   // the twiddles are there, and the previous polynomial's last reads of the exchange buffer are done

        // column half of the forward transform of each target, both lane halves at once (different moduli per half)
        double* lh = lds + h * HALF_WORDS;
#pragma unroll
        for (int u = 0; u < TL; ++u) {
            uint32_t tw_at = (h * TL + u) * TW_WORDS;
            asm volatile("" : "+v"(tw_at));   // they stay in LDS: hoisted out of the loop they take sixty registers a target
            const double* ta = lds_tw + tw_at;
            radix16_fwd(acc[u], *reinterpret_cast<const double(*)[16]>(ta), mt[u]);
            if constexpr (E > 0) {
                if (u > 0) __syncthreads();  // the previous target's reads of the exchange buffer are done
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const uint32_t row = r0 + S * k;
                    lh[row * TC + (row >> 4) * PADW + c] = acc[u][k];
                }
                __syncthreads();
#pragma unroll
                for (int k = 0; k < 16; ++k) acc[u][k] = lh[(16 * r0 + k) * TC + r0 * PADW + c];
                radix16_fwd<4 - E>(acc[u], *reinterpret_cast<const double(*)[16]>(ta + 16 * (1 + r0)), mt[u]);
            }
            if (tgt[u] < n_dst) packed_store<256>(out + (uint64_t)poly * out_ps + (uint64_t)dst_limb[u] * packed_limb_bytes(N), N, r0 * 1024 + col, pack(acc[u]));
            if (u == 0 && poly + step < n_polys) request(poly + step);
        }
    }
}

// ---- row half of the forward transform of the raised limbs + inner product with the key (see ks_fused.hip) ----------
// One wavefront: four rows (group rg) of limb position pos of one batch item.  d_b / lifted_b: that batch item's
// d [ell][N] words and raised digits [ndig][E] in packed limbs.
// What becomes of the two sums:
//   FINISH == 0: they are left in acc ([2][E] packed limbs).  Those of the ciphertext limbs stay there in rows order; those of the special
// limbs, and of limb ell - 1 where drop says that it is dropped (drop: that batch item's addend [2][ell], packed; null otherwise), go
// through the row half of their inverse transform and are left in columns order.
//   FINISH == 1 (ciphertext limbs): the division itself, out = (sum - conv) * mul, conv being the converted limbs [2][ell], whose forward row
// half is done here; FINISH == 2: + addend * admul (packed, [2][ell]).
// WD / WK: word types of d and of the key (64-bit, or 32-bit for moduli below 2^32; uint8_t: d in packed limbs, rows order); the output
// has the key's.
// PREFETCH: loads are requested in the order x(0), key(0), x(1), key(1), ... and return in that order.
// While digit j is transformed, key(j) and x(j + 1) are in flight; every key slot is refilled with the next digit's as soon
// as its product is done, so key(j + 1) has the whole transform of digit j + 1 to arrive.
struct InnerProductLds {
    double rows[4 * kRowPitch];        // exchange buffer
    double ta[4 * 16], tb[15 * 64];    // twiddles: every digit's transform uses the same ones (store_row_twiddles)
};
// What the sums of a task end in (see above).
template <typename W>
struct SumsEnd {
    uint8_t* acc;              // FINISH == 0
    const uint8_t* drop;
    double drop_mul;
    const uint8_t *conv, *addend;   // FINISH > 0
    W* out;                    // limb pos of component 0
    uint64_t out_comp;         // words to that of component 1
    double mul, admul;
};
template <int LOG_R, typename WD, typename WK, bool PREFETCH, int FINISH>
__device__ __forceinline__ void task_rows_inner_product(const TwTables& tw, const TwTables& twi, const Mod* __restrict__ mods,
                                                        const DigitRanges& dg, uint32_t ell, uint32_t E, uint32_t L, uint32_t M,
                                                        const WD* __restrict__ d_b, const uint8_t* __restrict__ lifted_b,
                                                        const WK* __restrict__ evk, const SumsEnd<WK>& end, uint32_t pos,
                                                        uint32_t rg, uint32_t lane, InnerProductLds& lds) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R;
    constexpr uint64_t LIMB = packed_limb_bytes(N);
    const uint32_t mid = pos < ell ? pos : L + (pos - ell);
    const Mod m = mods[mid];
    const uint32_t j0 = lane & 15, rr = lane >> 4, row = rg * 4 + rr;
    const uint32_t off = row * 256 + j0, at = rg * 256 + lane;
    double* lrow = lds.rows + rr * kRowPitch;
    double a0[16], a1[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) a0[k] = a1[k] = 0.0;

    // the digit's own limbs come in boundary words, the raised ones packed: two load shapes, so the (uniform) choice is a branch
    struct Source {
        uint32_t w[sizeof(WD) == 8 ? 32 : 20];   // 16 words, or a PackedRaw
    };
    const auto own = [&](uint32_t j) { return pos >= dg.lo[j] && pos < dg.hi[j]; };
    const auto request = [&](uint32_t j, Source& x) {
        if constexpr (sizeof(WD) == 1) {
            const PackedRaw t = packed_load<64>(own(j) ? d_b + pos * LIMB : lifted_b + ((uint64_t)j * E + pos) * LIMB, N, at);
#pragma unroll
            for (int k = 0; k < 16; ++k) x.w[k] = t.lo[k];
#pragma unroll
            for (int k = 0; k < 4; ++k) x.w[16 + k] = t.hi[k];
        } else if (own(j)) {
            const WD* src = d_b + (uint64_t)pos * N + off;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const WD t = src[16 * k];
                if constexpr (sizeof(WD) == 8) {
                    x.w[2 * k] = (uint32_t)t;
                    x.w[2 * k + 1] = (uint32_t)((uint64_t)t >> 32);
                } else {
                    x.w[k] = t;
                }
            }
            // Both branches write every entry: stores of 16 here and 20 there are merged into one with a variable index, which keeps the
            // array in scratch memory (28-bit key-switches, N = 2^16, 17 limbs: one 81.0 -> 79.4 us without it, 16 733 -> 715).
            if constexpr (sizeof(WD) == 4) {
#pragma unroll
                for (int k = 16; k < 20; ++k) x.w[k] = 0;
            }
        } else {
            const PackedRaw t = packed_load<64>(lifted_b + ((uint64_t)j * E + pos) * LIMB, N, at);
#pragma unroll
            for (int k = 0; k < 16; ++k) x.w[k] = t.lo[k];
#pragma unroll
            for (int k = 0; k < 4; ++k) x.w[16 + k] = t.hi[k];
        }
    };
    const auto values = [&](uint32_t j, const Source& s, double (&x)[16]) {
        if constexpr (sizeof(WD) == 1) {
            PackedRaw t;
#pragma unroll
            for (int k = 0; k < 16; ++k) t.lo[k] = s.w[k];
#pragma unroll
            for (int k = 0; k < 4; ++k) t.hi[k] = s.w[16 + k];
            if (own(j)) unpack(t, x);
            else unpack_rows(t, x);
        } else if (own(j)) {
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if constexpr (sizeof(WD) == 8) x[k] = word_to_f64<WD>((uint64_t)s.w[2 * k + 1] << 32 | s.w[2 * k]);
                else x[k] = word_to_f64<WD>(s.w[k]);
        } else {
            PackedRaw t;
#pragma unroll
            for (int k = 0; k < 16; ++k) t.lo[k] = s.w[k];
#pragma unroll
            for (int k = 0; k < 4; ++k) t.hi[k] = s.w[16 + k];
            unpack_rows(t, x);
        }
    };
    const auto transform = [&](double (&x)[16]) {
        uint32_t ta_at = rr * 16, tb_at = lane;
        asm volatile("" : "+v"(ta_at), "+v"(tb_at));   // the twiddles stay in LDS: hoisted out of the loop they take sixty registers
        radix16_fwd_lds(x, lds.ta + ta_at, 1, m);
#pragma unroll
        for (int k = 0; k < 16; ++k) lrow[j0 + 17 * k] = x[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = lrow[17 * j0 + k];
        radix16_fwd_lds(x, lds.tb + tb_at - 64, 64, m);
#pragma unroll
        for (int k = 0; k < 16; ++k) lrow[17 * j0 + k] = x[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = lrow[j0 + 17 * k];
    };
    const WK* keys = evk + (uint64_t)mid * N + off;
    const uint64_t comp = (uint64_t)M * N;
    Source xn;
    PackedRaw conv, addend;
    const auto request_end = [&](uint32_t comp) {
        conv = packed_load<64>(end.conv + ((uint64_t)comp * ell + pos) * LIMB, N, at);
        if constexpr (FINISH == 2) addend = packed_load<64>(end.addend + ((uint64_t)comp * ell + pos) * LIMB, N, at);
    };
    request(0, xn);
    store_row_twiddles(lds.ta, lds.tb, tw, mid, N, R + row, lane, m);
    __syncthreads();
    static_assert(PREFETCH || FINISH == 0, "built forms");
    if constexpr (PREFETCH) {
        WK kc0[16], kc1[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            kc0[k] = keys[16 * k];
            kc1[k] = keys[comp + 16 * k];
        }
        auto digit = [&](uint32_t j, auto next) {
            constexpr bool NEXT = decltype(next)::value;
            const WK* kp = keys + (uint64_t)(j + 1) * 2 * comp;
            double x[16];
            values(j, xn, x);
            if constexpr (NEXT) request(j + 1, xn);
            else if constexpr (FINISH != 0) request_end(0);
            if (!own(j)) transform(x);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                a0[k] += mulmod_lazy(x[k], word_to_f64<WK>(kc0[k]), m);
                a1[k] += mulmod_lazy(x[k], word_to_f64<WK>(kc1[k]), m);
                if constexpr (NEXT) {
                    kc0[k] = kp[16 * k];
                    kc1[k] = kp[comp + 16 * k];
                }
            }
        };
#pragma unroll 1
        for (uint32_t j = 0; j + 1 < dg.ndig; ++j) digit(j, std::true_type{});
        digit(dg.ndig - 1, std::false_type{});
    } else {
#pragma unroll 1
        for (uint32_t j = 0; j < dg.ndig; ++j) {
            const WK* kp = keys + (uint64_t)j * 2 * comp;
            // issue every load of this digit up front (the key slots are independent of the transform below)
            if (j != 0) request(j, xn);
            WK k0[16], k1[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) k0[k] = kp[16 * k];
#pragma unroll
            for (int k = 0; k < 16; ++k) k1[k] = kp[comp + 16 * k];
            double x[16];
            values(j, xn, x);
            if (!own(j)) transform(x);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                a0[k] += mulmod_lazy(x[k], word_to_f64<WK>(k0[k]), m);
                a1[k] += mulmod_lazy(x[k], word_to_f64<WK>(k1[k]), m);
            }
        }
    }
    if constexpr (FINISH != 0) {
        const auto finish = [&](const double (&a)[16], uint32_t comp) {
            double w[16], ad[16];
            unpack_rows(conv, w);
            if constexpr (FINISH == 2) unpack(addend, ad);
            if (comp == 0) request_end(1);   // ahead of the stores (loads and stores share one in-order counter)
            transform(w);
            WK* op = end.out + comp * end.out_comp + off;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                double r = mulmod_lazy(a[k] - w[k], end.mul, m);
                if constexpr (FINISH == 2) r = reduce_lazy(r + mulmod_lazy(ad[k], end.admul, m), m);
                op[16 * k] = f64_to_word<WK>(canon(r, m));
            }
        };
        finish(a0, 0);
        finish(a1, 1);
    } else {
        uint8_t* o0 = end.acc + (uint64_t)pos * LIMB;
        uint8_t* o1 = end.acc + ((uint64_t)E + pos) * LIMB;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            a0[k] = reduce_lazy(a0[k], m);
            a1[k] = reduce_lazy(a1[k], m);
        }
        const bool dropped = end.drop && pos + 1 == ell;  // uniform
        if (pos < ell && !dropped) {
            packed_store<64>(o0, N, at, pack(a0));
            packed_store<64>(o1, N, at, pack(a1));
            return;
        }
        if (dropped) {  // the limb a rescale drops becomes a source like the special limbs, its addend included
            const PackedRaw r0 = packed_load<64>(end.drop + (uint64_t)pos * LIMB, N, at), r1 = packed_load<64>(end.drop + ((uint64_t)ell + pos) * LIMB, N, at);
            double d0[16], d1[16];
            unpack(r0, d0);
            unpack(r1, d1);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                a0[k] = reduce_lazy(a0[k] + mulmod_lazy(d0[k], end.drop_mul, m), m);
                a1[k] = reduce_lazy(a1[k] + mulmod_lazy(d1[k], end.drop_mul, m), m);
            }
        }
        // Special limbs go straight into ModDown: the row half of their inverse transform works on the very
        // rows this wavefront holds, so it is done here and handed to the column half.
        PassTwiddles ti;
        load_row_twiddles(ti, twi, mid, N, R + row, j0, m);
        row_inv_core(a0, ti, j0, lrow, m);
        row_inv_core(a1, ti, j0, lrow, m);
        packed_store<64>(o0, N, at, pack_rows(a0));
        packed_store<64>(o1, N, at, pack_rows(a1));
    }
}

// ---- the same (FINISH == 0) for launches of few wavefronts: a workgroup per four rows, a wavefront per digit and one per key component ----
// A wavefront of task_rows_inner_product works through its digits one after the other (load, transform, products) and then through both
// components; where a launch leaves the chip idle that chain is its time.  Here every load of the four rows is requested at once:
// wavefront j < ndig transforms digit j and leaves it in LDS, wavefront ndig + c multiplies by the keys of component c, adds and does
// what follows for that component.
// Every wavefront passes the same three barriers: twiddles ready, digits ready, digits read.
// lds: rows_split_lds(ndig) bytes.
struct RowTwiddlesLds {
    double ta[4 * 16], tb[15 * 64];
};
constexpr uint32_t kRowsBuffer = 4 * kRowPitch;   // doubles: four rows of an exchange buffer
constexpr uint32_t rows_split_lds(uint32_t ndig) {
    return (ndig < 2 ? 2 : ndig) * kRowsBuffer * 8 + 2 * (uint32_t)sizeof(RowTwiddlesLds);
}
template <int LOG_R, typename WD, typename WK>
__device__ __forceinline__ void task_rows_split(const TwTables& tw, const TwTables& twi, const Mod* __restrict__ mods, const DigitRanges& dg,
                                                uint32_t ell, uint32_t E, uint32_t L, uint32_t M, const WD* __restrict__ d_b,
                                                const uint8_t* __restrict__ lifted_b, const WK* __restrict__ evk, const SumsEnd<WK>& end,
                                                uint32_t pos, uint32_t rg, uint32_t wave, uint32_t lane, double* lds) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R;
    constexpr uint64_t LIMB = packed_limb_bytes(N);
    const uint32_t mid = pos < ell ? pos : L + (pos - ell);
    const Mod m = mods[mid];
    const uint32_t j0 = lane & 15, rr = lane >> 4, row = rg * 4 + rr;
    const uint32_t off = row * 256 + j0, at = rg * 256 + lane;
    RowTwiddlesLds* tf = reinterpret_cast<RowTwiddlesLds*>(lds);   // forward, then inverse
    RowTwiddlesLds* ti = tf + 1;
    double* rows = reinterpret_cast<double*>(tf + 2);
    const bool dropped = end.drop && pos + 1 == ell, divided = pos >= ell || dropped;   // uniform
    if (wave < dg.ndig) {
        const uint32_t j = wave;
        const bool own = pos >= dg.lo[j] && pos < dg.hi[j];   // uniform
        double* lrow = rows + j * kRowsBuffer + rr * kRowPitch;
        double x[16];
        if (own) {
            if constexpr (sizeof(WD) == 1) {
                const PackedRaw t = packed_load<64>(reinterpret_cast<const uint8_t*>(d_b) + pos * LIMB, N, at);
                unpack(t, x);
            } else {
                const WD* src = d_b + (uint64_t)pos * N + off;
#pragma unroll
                for (int k = 0; k < 16; ++k) x[k] = word_to_f64<WD>(src[16 * k]);
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) lrow[j0 + 17 * k] = x[k];
            __syncthreads();
        } else {
            const PackedRaw t = packed_load<64>(lifted_b + ((uint64_t)j * E + pos) * LIMB, N, at);
            __syncthreads();
            unpack_rows(t, x);
            radix16_fwd_lds(x, tf->ta + rr * 16, 1, m);
#pragma unroll
            for (int k = 0; k < 16; ++k) lrow[j0 + 17 * k] = x[k];
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = lrow[17 * j0 + k];
            radix16_fwd_lds(x, tf->tb + lane - 64, 64, m);
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < 16; ++k) lrow[17 * j0 + k] = x[k];
        }
        __syncthreads();
        __syncthreads();
        return;
    }
    const uint32_t c = wave - dg.ndig;
    const uint64_t comp = (uint64_t)M * N;
    const WK* keys = evk + (uint64_t)mid * N + off + c * comp;
    // keys requested ahead of everything else; the others follow when these are used
    constexpr uint32_t AHEAD = 2;
    WK key[AHEAD][16];
#pragma unroll
    for (uint32_t a = 0; a < AHEAD; ++a) {
        const WK* kp = keys + (uint64_t)min(a, dg.ndig - 1) * 2 * comp;
#pragma unroll
        for (int k = 0; k < 16; ++k) key[a][k] = kp[16 * k];
    }
    if (c == 1 || divided) {
        const TwTables t{c ? tw.W : twi.W, c ? tw.trow : twi.trow, c ? tw.w16 : twi.w16};
        RowTwiddlesLds* to = c ? tf : ti;
        store_row_twiddles(to->ta, to->tb, t, mid, N, R + row, lane, m);
    }
    __syncthreads();
    __syncthreads();
    double a[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) a[k] = 0.0;
#pragma unroll 1
    for (uint32_t j = 0; j < dg.ndig; j += AHEAD) {
        if (j != 0) {
#pragma unroll
            for (uint32_t i = 0; i < AHEAD; ++i) {
                const WK* kp = keys + (uint64_t)min(j + i, dg.ndig - 1) * 2 * comp;
#pragma unroll
                for (int k = 0; k < 16; ++k) key[i][k] = kp[16 * k];
            }
        }
#pragma unroll
        for (uint32_t i = 0; i < AHEAD; ++i) {
            if (j + i >= dg.ndig) break;
            const double* x = rows + (j + i) * kRowsBuffer + rr * kRowPitch + j0;
#pragma unroll
            for (int k = 0; k < 16; ++k) a[k] += mulmod_lazy(x[17 * k], word_to_f64<WK>(key[i][k]), m);
        }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) a[k] = reduce_lazy(a[k], m);
    __syncthreads();   // both components have read the digits: their buffers are free
    uint8_t* out = end.acc + ((uint64_t)c * E + pos) * LIMB;
    if (!divided) {
        packed_store<64>(out, N, at, pack(a));
        return;
    }
    double* lrow = rows + c * kRowsBuffer + rr * kRowPitch;
    if (dropped) {
        double ad[16];
        unpack(packed_load<64>(end.drop + ((uint64_t)c * ell + pos) * LIMB, N, at), ad);
#pragma unroll
        for (int k = 0; k < 16; ++k) a[k] = reduce_lazy(a[k] + mulmod_lazy(ad[k], end.drop_mul, m), m);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) lrow[j0 + 17 * k] = a[k];
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 16; ++k) a[k] = lrow[17 * j0 + k];
    radix16_inv_lds(a, ti->tb + lane - 64, 64, m);
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 16; ++k) lrow[17 * j0 + k] = reduce_lazy(a[k], m);
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 16; ++k) a[k] = lrow[j0 + 17 * k];
    radix16_inv_lds(a, ti->ta + rr * 16, 1, m);
#pragma unroll
    for (int k = 0; k < 16; ++k) a[k] = reduce_lazy(a[k], m);
    packed_store<64>(out, N, at, pack_rows(a));
}

// ---- row half of the forward transform of the converted limbs + (acc - conv) * mul (+ addend) ------------------------
// One wavefront: four rows (group rg) of limb i.  conv / acc: that limb of the converted limbs and of the accumulators, packed; op: of the
// output.  adp: that limb of the addend.  ADDEND: 0 = none, 1 = words like the output's, read through sigma_galois where GATHER,
// added as they are, 2 = packed, multiplied by admul first.
template <int LOG_R, bool GATHER, int ADDEND, typename W>
__device__ __forceinline__ void task_rows_finish(const TwTables& tw, Mod m, uint32_t mod_id, double mul, double admul,
                                                 const uint8_t* __restrict__ conv, const uint8_t* __restrict__ acc, W* __restrict__ op,
                                                 const void* __restrict__ adp, uint32_t galois, uint32_t rg, uint32_t lane, double* lds_wave) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R, LOGN = LOG_R + 8;
    const uint32_t j0 = lane & 15, rr = lane >> 4, row = rg * 4 + rr;
    const uint32_t off = row * 256 + j0, at = rg * 256 + lane;
    // issue every load up front: the accumulator (and addend) slots do not depend on the transform
    const PackedRaw wr = packed_load<64>(conv, N, at), ar = packed_load<64>(acc, N, at);
    PackedRaw dr;
    W dw[16];
    if constexpr (ADDEND == 2) {
        dr = packed_load<64>(static_cast<const uint8_t*>(adp), N, at);
    } else if constexpr (ADDEND == 1) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t n = off + 16 * k;
            dw[k] = static_cast<const W*>(adp)[GATHER ? galois_source_slot(n, galois, LOGN) : n];
        }
    }
    PassTwiddles t;
    load_row_twiddles(t, tw, mod_id, N, R + row, j0, m);
    double w[16], a[16], ad[16];
    unpack_rows(wr, w);
    row_fwd_core(w, t, j0, lds_wave + rr * kRowPitch, m);
    unpack(ar, a);
    if constexpr (ADDEND == 2) unpack(dr, ad);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        double r = mulmod_lazy(a[k] - w[k], mul, m);
        if constexpr (ADDEND == 1) r = reduce_lazy(r + word_to_f64<W>(dw[k]), m);
        if constexpr (ADDEND == 2) r = reduce_lazy(r + mulmod_lazy(ad[k], admul, m), m);
        op[off + 16 * k] = f64_to_word<W>(canon(r, m));
    }
}

}  // namespace ks
