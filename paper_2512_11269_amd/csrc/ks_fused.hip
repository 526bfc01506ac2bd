// Vertically fused kernels of the key-switching chain (the paper's vertical fusion: dependent limb
// operations on the same positions stay in registers instead of making a round trip through memory).
//
//  * bconv_ntt_cols       base conversion of a digit feeding the column half of the forward transform of
//                         each target limb: the converted limb never exists in memory in coefficient form.
//  * rows_inner_product   row half of the forward transform of every raised limb feeding the inner product
//                         with the key: the raised limb never exists in memory in evaluation form.
//  * rows_moddown_finish  row half of the forward transform of the converted special part feeding
//                         (acc - conv) * P^-1 (+ addend).
//
// Base conversion is coefficient-wise and the column half touches a fixed set of coefficient positions per
// tile, so the first fusion is legal; the inner product and the final scale are slot-wise and the row half
// produces complete slots, so the other two are.
#include "ks_internal.hpp"
#include "ks_tasks.hpp"

namespace ks {

// One source of a conversion: acc[t][k] += y[k] * f[t] as exact integers -- each source point is split once (split3, or
// split2 when every modulus is below 2^32), every target adds PIECES products against its shifted, centred factors.
// REFILL: once y[k] has been consumed, the same registers receive point k of the next source (byte offset next_off in
// the buffer), which then has a whole source's worth of arithmetic to arrive.
// The factors of the next source (fnext: uniform, scalar loads) are requested after the first point, together with
// the limb index of the source after next: scalar loads complete out of order, so the first use of f waits for every
// scalar load in flight, and at that moment only f's own, requested a source ago, should be.
template <int LOG_R, int TS, bool REFILL, int PIECES>
__device__ __forceinline__ void bconv_accumulate(double (&acc)[TS][16], double (&y)[16], const double (&f)[TS][3],
                                                 double (&fnext)[TS][3], const double* const (&hat_row)[TS], int inext,
                                                 uint32_t& limb_after, const uint32_t* src_limb, int iafter, BufferRsrc rsrc,
                                                 uint32_t lane_off, uint32_t next_off) {
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        double y2 = 0.0, y1, y0;
        if constexpr (PIECES == 3) split3(y[k], y2, y1, y0);
        else split2(y[k], y1, y0);
        if (REFILL) y[k] = load_strided_point<LOG_R>(rsrc, lane_off, next_off, k);
#pragma unroll
        for (int tt = 0; tt < TS; ++tt) {
            acc[tt][k] = __builtin_fma(y1, f[tt][1], __builtin_fma(y0, f[tt][0], acc[tt][k]));
            if constexpr (PIECES == 3) acc[tt][k] = __builtin_fma(y2, f[tt][2], acc[tt][k]);
        }
        if (k == 0) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int tt = 0; tt < TS; ++tt)
#pragma unroll
                for (int p = 0; p < PIECES; ++p) fnext[tt][p] = hat_row[tt][inext * 4 + p];
            limb_after = src_limb[iafter];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // one refill per point, in order, each after a point's worth of arithmetic: the wait before point k then leaves 15
    // loads in flight, while the arithmetic of neighbouring points may still interleave
    if (REFILL) {
#pragma unroll
        for (int k = 1; k < 16; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x002, PIECES == 3 ? 6 + 3 * TS : 3 + 2 * TS, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// y: [poly][..][N] canonical doubles y_i = [x_i N^-1 (D/s_i)^-1]_{s_i} (written by ntt_inv_cols with its
// scale table).  Each workgroup owns one column tile (4096 positions) and TS targets of one digit: it
// accumulates sum_i y_i * (D/s_i mod t) as an exact integer (split3) for its 16 positions per thread, then runs the
// column stages of the forward transform modulo t and stores raw doubles.  The sources are re-read by the workgroups of
// the other target subsets; those reads are served by L2 / the last-level cache.
// ------------------------------------------------------------------------------------------------
// PIECES: 3 in general (moduli below 2^36); 2 when every modulus of the context is below 2^32 (the plan's factors are
// then cut at 16 bits: two products per source and target instead of three).
template <int LOG_R, int TS, bool TWO_SETS, int PIECES>
__global__ __launch_bounds__(256) void bconv_ntt_cols(const double* __restrict__ tw, const BConvPlan* __restrict__ plans,
                                                      const uint64_t* __restrict__ y, uint64_t y_ps, uint64_t* __restrict__ out,
                                                      uint64_t out_ps, uint32_t n_subsets) {
    constexpr uint32_t N = 256u << LOG_R, TILES = 1u << (LOG_R - 4), TC = 256 / TILES;
    __shared__ double lds[LOG_R > 4 ? 4096 : 1];
    const uint32_t tid = threadIdx.x, tile = blockIdx.x;
    const uint32_t plan_id = blockIdx.y / n_subsets, subset = blockIdx.y - plan_id * n_subsets;
    const BConvPlan& P = plans[plan_id];
    const int n_dst = (int)P.n_dst, n_src = (int)P.n_src;
    const int t0 = (int)subset * TS;
    if (t0 >= n_dst) return;  // uniform for the whole workgroup
    const uint64_t* yp = y + (uint64_t)blockIdx.z * y_ps;
    uint64_t* op = out + (uint64_t)blockIdx.z * out_ps;
    const uint32_t c = tid & (TC - 1), r0 = tid / TC, col = tile * TC + c;

    double acc[TS][16];
#pragma unroll
    for (int tt = 0; tt < TS; ++tt)
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[tt][k] = 0.0;

    // Per-target constants.  They are uniform across the workgroup and travel through scalar loads.
    Mod mt[TS];
    const double* hat_row[TS];
#pragma unroll
    for (int tt = 0; tt < TS; ++tt) {
        const int t = min(t0 + tt, n_dst - 1);  // a ragged last subset recomputes its last target (stored once)
        mt[tt] = P.dst_mod[t];
        hat_row[tt] = &P.hats[t][0][0];
    }

    // Software pipeline over the sources, two per trip so that the uniform factors can alternate between two scalar
    // register sets, with the limb index of the source after next fetched ahead as well: nothing is waited for right
    // after it was requested.  The 16 points of a source are either held in ONE register set that is refilled point by
    // point with the next source while it is consumed (fewer registers; best for the few-workgroup launches of a single
    // ciphertext), or in TWO sets, the idle one filled by a burst of 16 loads (measured 6 % faster on full-chip launches).
    // Sources past the end are zero-padded in the plan (factor 0, a valid limb): prefetches are unconditional -- a
    // conditional one would make the wait-count bookkeeping assume the worst at the join and stall every use on the
    // newest loads -- and an odd source count simply runs one padding source.  Loads are fenced into use order, before
    // the loop as inside it, so that every wait leaves exactly the younger loads in flight.  The points are read through a
    // buffer descriptor of this polynomial's bundle: per-lane offset in a vector register, limb and row offset in a
    // scalar one, so switching limb costs no vector instructions.
    const BufferRsrc ysrd = make_buffer_rsrc(yp, y_ps * 8);
    const uint32_t lane_off = (r0 * 256 + col) * 8;
    double yv[16], ha[TS][3], hb[TS][3];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        yv[k] = load_strided_point<LOG_R>(ysrd, lane_off, P.src_limb[0] * (N * 8), k);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int tt = 0; tt < TS; ++tt)
#pragma unroll
        for (int p = 0; p < PIECES; ++p) ha[tt][p] = hat_row[tt][p];
    uint32_t limb_next = P.src_limb[1];

    if constexpr (!TWO_SETS) {
#pragma unroll 1
        for (int i = 0; i < n_src; i += 2) {
            uint32_t limb_after;
            bconv_accumulate<LOG_R, TS, true, PIECES>(acc, yv, ha, hb, hat_row, min(i + 1, kMaxSrc - 1), limb_after, P.src_limb,
                                              min(i + 2, kMaxSrc - 1), ysrd, lane_off, limb_next * (N * 8));
            bconv_accumulate<LOG_R, TS, true, PIECES>(acc, yv, hb, ha, hat_row, min(i + 2, kMaxSrc - 1), limb_next, P.src_limb,
                                              min(i + 3, kMaxSrc - 1), ysrd, lane_off, limb_after * (N * 8));
        }
    } else {
        double yw[16];
#pragma unroll 1
        for (int i = 0; i < n_src; i += 2) {
            uint32_t limb_after;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                yw[k] = load_strided_point<LOG_R>(ysrd, lane_off, limb_next * (N * 8), k);
                __builtin_amdgcn_sched_barrier(0);
            }
            bconv_accumulate<LOG_R, TS, false, PIECES>(acc, yv, ha, hb, hat_row, min(i + 1, kMaxSrc - 1), limb_after, P.src_limb,
                                               min(i + 2, kMaxSrc - 1), ysrd, lane_off, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                yv[k] = load_strided_point<LOG_R>(ysrd, lane_off, limb_after * (N * 8), k);
                __builtin_amdgcn_sched_barrier(0);
            }
            bconv_accumulate<LOG_R, TS, false, PIECES>(acc, yw, hb, ha, hat_row, min(i + 2, kMaxSrc - 1), limb_next, P.src_limb,
                                               min(i + 3, kMaxSrc - 1), ysrd, lane_off, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // Twiddles are requested one target ahead and always before the previous target's stores are issued: loads and
    // stores share one in-order counter, so a wait for a load issued after a store would also wait for the store to be
    // acknowledged by memory.
    PassTwiddles tws;
    load_col_twiddles<LOG_R>(tws, tw + (size_t)P.dst_mod_id[t0] * N, r0);
#pragma unroll
    for (int tt = 0; tt < TS; ++tt) {
        const int t = t0 + tt;
        if (t < n_dst) {  // uniform
            PassTwiddles cur = tws;
            if (tt + 1 < TS && t + 1 < n_dst) load_col_twiddles<LOG_R>(tws, tw + (size_t)P.dst_mod_id[t + 1] * N, r0);
#pragma unroll
            for (int k = 0; k < 16; ++k) acc[tt][k] = reduce_lazy(acc[tt][k], mt[tt]);
            col_fwd_core<LOG_R>(acc[tt], cur, c, r0, lds, mt[tt]);
            uint64_t* dst = op + (uint64_t)P.dst_limb[t] * N;
#pragma unroll
            for (int k = 0; k < 16; ++k) store_f64(dst + col_row_grouped<LOG_R>(r0, k) * 256 + col, acc[tt][k]);
            if constexpr (LOG_R > 4) __syncthreads();  // the exchange buffer is reused by the next target
        }
    }
}

// Which kernel the two conversions of a call take: 0 vector, 8 or 16 matrix cores with tiles of 8 or 16 columns.  One answer
// for both: the code of a kernel that ran a moment ago is still in the caches, so a call that mixes them pays 1-2 us at
// small sizes and 5-8 where its data exceed the memory-side cache (three key-switches 8 -> 3 x 24 and 8 -> 24, N = 2^16,
// 36-bit: vector 248 us, matrix cores in ModUp only 246, in ModDown only 242, in both 230).
//   G counts the matrix-core kernel's workgroups, six targets and 2048 positions each, of which 512 run at once.  Their cost
// hardly depends on the sources; the vector kernel takes one instruction per source and piece of a residue (three pieces,
// two for moduli below 2^32) and some for the transform.  So the line is drawn by the load, the vector instructions that a
// group of six targets replaces, 20 per target besides the products: many sources and full groups (20 targets take four, 24
// too) favour the matrix cores.  The lines come from key-switches of 42 parameter sets, 1 to 8 ciphertexts, and hoisted
// rotations of 20, in both word sizes with every pair of kernels.  Times of calls in us, vector / 8 columns / 16 columns:
//   N = 2^16, 36-bit moduli.  4 -> 16 (load 171), 6 ciphertexts: 305 / 314; 5 -> 20 (175), 2: 169 / 157, 4: 280 / 274;
// 8 -> 24 (264), 1: 103 / 98, 4: 302 / 287; 12 -> 36 (336), 2: 272 / 241.  28-bit: 4 -> 16 (149), 6: 264 / 279; 8 -> 24
// (216), 2: 155 / 145, 7: 425 / 416.  In a single round one workgroup's chain is what counts, so the sources alone decide:
// 36-bit 4 -> 12 70 / 71, 5 -> 5 58 / 56, 7 -> 7 63 / 60, 10 -> 20 91 / 87; 28-bit 7 -> 7 58 / 59, 10 -> 20 82 / 83,
// 12 -> 18 84 / 84.
//   16 columns are whole lines, but one workgroup of 512 threads per compute unit that works in step: ahead when a launch
// has six rounds or more.  8 -> 24, 8 ciphertexts (G = 3072): 550 / 545 / 546; 12 -> 36 (4608): 906 / 903 / 887; four
// rotations of them (G of ModDown 8192 and 12288): 1663 / 1697 / 1614 and 2685 / 2730 / 2618, 28-bit 1492 / 1547 / 1464 and
// 2423 / 2508 / 2379 (8 -> 24 has a load of 216 there), but at G = 3456 582 / 587 / 585.  10 -> 20 (250), whose last group of six is mostly empty:
// 1477 / 1580 / 1497, hence the fill.
//   N = 2^15, 36-bit: 3 -> 9 (130), 8 ciphertexts: 123 / 120, 7: +3.5 %; 7 -> 21 (215), 4: 158 / 139; 28-bit: 3 -> 9 (117),
// 7: +5.6 %; 4 -> 12 (168), 4: 82 / 83, 8: 137 / 132; 5 -> 20 (150), 4: 140 / 133.  Where a launch has just more than 256 or
// 512 workgroups a few compute units do twice the work of the others: 3 -> 9, 3: 70 / 74; 13 -> 13 (256), 6: 130 / 134.
//   Below N = 2^15 launches are at their floor and the vector kernel is 0-1 us ahead.
int conversion_tile(const ks_ctx* c, const PlanSet& up, uint32_t up_polys, const PlanSet& down, uint32_t down_polys) {
    if (c->logN < 15) return 0;
    const uint64_t tiles = c->N / 2048, g_up = tiles * up.sixes * up_polys, g_down = tiles * down.sixes * down_polys;
    const uint64_t sixes = up.sixes + 2 * down.sixes, targets = up.targets + 2 * down.targets;
    const uint64_t load = 20 * targets + c->pieces * (up.products + 2ull * down.products);   // of one ciphertext
    const bool two_pieces = c->pieces == 2;
    const auto uneven = [](uint64_t g) { return (g > 256 && g <= 300) || (g > 512 && g <= 600); };
    const uint64_t extra = uneven(g_up) || uneven(g_down) ? 45 : 0;
    if (c->logN == 15) return load >= (extra + (two_pieces && g_up + g_down <= 1024 ? 160 : 132)) * sixes ? 8 : 0;
    if (g_up + g_down <= 512) return load >= (two_pieces ? 44 : 35) * targets ? 8 : 0;   // sources x pieces of 24 or 15
    if (std::max(g_up, g_down) < 3072) return load >= (extra + 173) * sixes ? 8 : 0;
    const bool full = targets * 10 >= sixes * 54;
    return full && load >= 216 * sixes && (!two_pieces || std::max(g_up, g_down) >= 4096) ? 16 : 0;
}

void launch_bconv_ntt_cols(const ks_ctx* c, const PlanSet& plans, uint32_t limbs_moved_per_poly, const uint64_t* y, uint64_t y_ps,
                           uint64_t* out, uint64_t out_ps, uint32_t n_polys, int tile, hipStream_t s, double ops_per_coeff) {
    const uint32_t n_plans = plans.n_plans, max_targets = plans.max_targets;
    const BConvPlan* d_plans = plans.d_plans;
    if (n_polys == 0 || n_plans == 0) return;
    const int kernel = c->opt[KS_OPT_BCONV_KERNEL] ? c->opt[KS_OPT_BCONV_KERNEL] : (tile ? 2 : 1);
    if (kernel == 2) {
        // algorithmic fp64 / integer vector work per coefficient of this kernel: per target 9 to recombine and reduce the
        // five sums and 35 for the column half; per source 2 to cut it into bytes (the contraction itself runs on the
        // matrix cores: 25 int8 multiply-adds per source and target)
        double vec_ops = 0.0;
        for (uint32_t j = 0; j < n_plans; ++j) vec_ops += plans.meta.plan[j].n_dst * 44.0 + plans.shape_src * 2.0;
        ProfScope ps("bconv_mfma_ntt_cols", (double)limbs_moved_per_poly * n_polys * c->N * 8.0, s, vec_ops * n_polys * c->N);
        const int tl = c->opt[KS_OPT_BCONV_TARGETS] >= 1 && c->opt[KS_OPT_BCONV_TARGETS] <= 3 ? c->opt[KS_OPT_BCONV_TARGETS] : 3;
        launch_bconv_mfma_ntt_cols(c, plans, y, y_ps, out, out_ps, n_polys, tl, tile == 16, s);
        return;
    }
    // Targets per workgroup: fewer targets = more workgroups but more re-reads and re-splits of the sources.  Four (with
    // the two-set source pipeline) is best once the launch has a few workgroups per compute unit; for the
    // single-ciphertext launches three (one-set pipeline) measured best (384 and 256 workgroups: every one resident at
    // once, none waiting for a slot to free up).
    // The context option KS_OPT_BCONV_TARGETS overrides the choice.
    const uint32_t tiles = 1u << (c->logN - 12);
    int ts = (uint64_t)tiles * n_plans * ((max_targets + 3) / 4) * n_polys >= 512 ? 4 : 3;
    if (c->opt[KS_OPT_BCONV_TARGETS] >= 1 && c->opt[KS_OPT_BCONV_TARGETS] <= 4) ts = c->opt[KS_OPT_BCONV_TARGETS];
    if (c->logN != 16 && ts < 3) ts = 3;  // the other ring degrees come with the two production shapes only
    const uint32_t n_subsets = (max_targets + ts - 1) / ts;
    const dim3 grid(tiles, n_plans * n_subsets, n_polys), block(256);
    ProfScope ps("bconv_ntt_cols", (double)limbs_moved_per_poly * n_polys * c->N * 8.0, s, ops_per_coeff * n_polys * c->N);
#define KS_LAUNCH_BCONV(LOGR, TSV)                                                                                                      \
    if (c->pieces == 2)                                                                                                                 \
        hipLaunchKernelGGL((bconv_ntt_cols<LOGR, TSV, (TSV == 4), 2>), grid, block, 0, s, c->d_tw_fwd, d_plans, y, y_ps, out, out_ps,  \
                           n_subsets);                                                                                                  \
    else                                                                                                                                \
        hipLaunchKernelGGL((bconv_ntt_cols<LOGR, TSV, (TSV == 4), 3>), grid, block, 0, s, c->d_tw_fwd, d_plans, y, y_ps, out, out_ps,  \
                           n_subsets)
    if (c->logN == 16) {
        if (ts == 4) { KS_LAUNCH_BCONV(8, 4); }
        else if (ts == 3) { KS_LAUNCH_BCONV(8, 3); }
        else if (ts == 2) { KS_LAUNCH_BCONV(8, 2); }
        else { KS_LAUNCH_BCONV(8, 1); }
    } else {
#define KS_LAUNCH(LOGR)                        \
    if (ts == 4) { KS_LAUNCH_BCONV(LOGR, 4); } \
    else { KS_LAUNCH_BCONV(LOGR, 3); }
        KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
    }
#undef KS_LAUNCH_BCONV
}

// ------------------------------------------------------------------------------------------------
// acc[b][c][pos] = sum_j d~_j[pos] * key[j][c][m(pos)].  For pos inside digit j, d~_j[pos] is the input limb
// itself; otherwise it is the raised limb, whose row half of the forward transform is done here.
// One wavefront = four rows of one limb position; it walks the digits, so d~ is read once and feeds both key
// components (load reuse), and the accumulators are reduced and written once.
// ------------------------------------------------------------------------------------------------
// WD / WK: word types of d and of the key (64-bit, or 32-bit for moduli below 2^32).
template <int LOG_R, typename WD, typename WK, bool PREFETCH>
__global__ __launch_bounds__(64, PREFETCH ? 2 : 0) void rows_inner_product(TwTables tw, TwTables twi,
                                                         const Mod* __restrict__ mods, DigitRanges dg,
                                                         uint32_t ell, uint32_t E, uint32_t L, uint32_t M,
                                                         const WD* __restrict__ d, uint64_t d_ps,
                                                         const uint64_t* __restrict__ lifted, const WK* __restrict__ evk,
                                                         uint64_t* __restrict__ acc, uint32_t* __restrict__ accq_lo,
                                                         uint8_t* __restrict__ accq_hi, const uint32_t* __restrict__ drop_lo,
                                                         const uint8_t* __restrict__ drop_hi, double drop_mul,
                                                         uint32_t packed_limbs, uint32_t batch, uint32_t special_first) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R;
    __shared__ double lds[4 * kRowPitch];
    __shared__ double lds_ta[4 * 16];
    // Workgroup -> (row group, limb position, batch item).  Consecutive workgroup ids go to the eight XCDs in
    // turn, each with its own L2; the ids that land on one XCD walk through all batch items of one
    // (row group, position) tile before moving to the next tile, so the key slots and twiddles of a tile are
    // fetched into that L2 once and reused by the whole batch.
    const uint32_t slot = blockIdx.x >> 3, b = slot % batch, tile = (slot / batch) * 8 + (blockIdx.x & 7);
    if (tile >= (R / 4) * E) return;  // uniform: padding workgroups when the tile count is not a multiple of 8
    // special_first (launches whose wavefronts are all resident at once, i.e. a single ciphertext): the special limbs take
    // the first workgroup ids.  Their wavefronts have the most arithmetic after their last load (one more transform and the
    // two inverse row passes) and the memory system serves the earliest requests first, so started last they are the tail
    // of the launch (59 k cycles per special wavefront against 37 k for the others; 40.2 -> 37.1 us per launch).  Batched
    // launches keep them last: the next kernel reads exactly these limbs and finds them cached (0.5-2 % per call).
    const uint32_t rg = tile % (R / 4), slot_pos = tile / (R / 4), n_special = E - ell;
    const uint32_t pos = !special_first ? slot_pos : slot_pos < n_special ? ell + slot_pos : slot_pos - n_special;
    task_rows_inner_product<LOG_R, WD, WK, PREFETCH>(tw, twi, mods, dg, ell, E, L, M, d + (uint64_t)b * d_ps, lifted + (uint64_t)b * dg.ndig * E * N, evk,
                                      acc + (uint64_t)b * 2 * E * N, accq_lo + (uint64_t)b * 2 * ell * N,
                                      accq_hi + (uint64_t)b * 2 * ell * N, drop_lo + (uint64_t)b * 2 * ell * N,
                                      drop_hi + (uint64_t)b * 2 * ell * N, drop_mul, packed_limbs, pos, rg, threadIdx.x, lds, lds_ta);
}

void launch_rows_inner_product(const ks_ctx* c, const Level& lv, const void* d, uint64_t d_ps, const uint64_t* lifted,
                               const void* evk, uint64_t* acc, uint32_t batch, hipStream_t s, bool d_words32, bool key_words32,
                               const PackedDigits& accq, const PackedDigits* drop_addend) {
    if (batch == 0) return;
    const uint32_t packed_limbs = drop_addend ? lv.ell - 1 : lv.ell;
    const PackedDigits drop = drop_addend ? *drop_addend : accq;  // never read without a dropped limb
    DigitRanges dg;
    dg.ndig = lv.ndig;
    for (uint32_t j = 0; j < kMaxDigits; ++j) {
        dg.lo[j] = j < lv.ndig ? lv.digit_lo[j] : 0;
        dg.hi[j] = j < lv.ndig ? lv.digit_hi[j] : 0;
    }
    // reads: every raised digit limb per ciphertext and the key (once per call); writes: both accumulators
    // d (ell limbs per ciphertext) and the key arrive in boundary words, the raised limbs and the sums in 8 bytes
    const double wd = d_words32 ? 0.5 : 1.0, wk = key_words32 ? 0.5 : 1.0;
    ProfScope ps("rows_inner_product",
                 ((double)batch * ((lv.ndig * lv.E - lv.ell) + wd * lv.ell + 2.0 * lv.E - 0.75 * packed_limbs) + wk * 2.0 * lv.ndig * lv.E) *
                     c->N * 8.0,
                 s);
    const uint32_t tiles = (c->N / 1024) * lv.E;
    const dim3 grid(((tiles + 7) / 8) * 8 * batch), block(64);
    // launches with more than two wavefronts per SIMD (1024 SIMDs) to run take the variant that requests the next digit's
    // loads early: 3 % faster there (32.1 -> 31.0 us per multiplication at L = 35); the single-ciphertext launch is bound by
    // bandwidth and gains nothing from it
    const bool prefetch = grid.x > 2048;
#define KS_LAUNCH_IP(LOGR, WDT, WKT, PF)                                                                                           \
    hipLaunchKernelGGL((rows_inner_product<LOGR, WDT, WKT, PF>), grid, block, 0, s, c->tw_fwd, c->tw_inv, c->d_mod, dg, lv.ell, lv.E, c->L, \
                       c->M, static_cast<const WDT*>(d), d_ps, lifted, static_cast<const WKT*>(evk), acc, accq.lo, accq.hi, drop.lo, drop.hi,       \
                       lv.Pmod_last, packed_limbs, batch, prefetch ? 0u : 1u)
#define KS_LAUNCH(LOGR)                                                          \
    if (d_words32 && key_words32) KS_LAUNCH_IP(LOGR, uint32_t, uint32_t, false); \
    else if (key_words32) KS_LAUNCH_IP(LOGR, uint64_t, uint32_t, false);         \
    else if (prefetch) KS_LAUNCH_IP(LOGR, uint64_t, uint64_t, true);             \
    else KS_LAUNCH_IP(LOGR, uint64_t, uint64_t, false)
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_IP
}

// ------------------------------------------------------------------------------------------------
// out[b][comp][i] = (acc[b][comp][i] - NTT_rows(conv[b][comp][i])) * P^-1 (+ addend), canonical.
// ------------------------------------------------------------------------------------------------
// ADDEND: 0 = none, 1 = added as it is, 2 = multiplied by addend_mul[i] first.  Compile-time so that the kernel has no
// branch: behind a run-time test every addend load became its own load-wait-use round trip.  A launch covers the
// components comp0 .. comp0 + n_comps - 1 of every batch item.
// ACCP: the ciphertext limbs of the accumulator come packed (acc: [b][2][ell][N] 32-bit low words, acc_hi: the bytes
// above) instead of as the first ell limbs of [b][2][E][N] 64-bit words.
// ADF: format of the addend: 0 = 64-bit words; 1 = packed the same way (addend: [b][2][ell][N] low words, addend_hi: the
// bytes above); 2 = 32-bit words.
template <int LOG_R, bool GATHER, int ADDEND, typename W, bool ACCP, int ADF>
__global__ __launch_bounds__(64) void rows_moddown_finish(TwTables tw, const Mod* __restrict__ mods,
                                                          const double* __restrict__ Pinv, const double* __restrict__ addend_mul,
                                                          uint32_t ell, uint32_t E, uint32_t out_limbs,
                                                          const void* __restrict__ acc, const uint8_t* __restrict__ acc_hi,
                                                          const uint64_t* __restrict__ conv,
                                                          W* __restrict__ out, uint64_t out_bs,
                                                          const void* __restrict__ addend, const uint8_t* __restrict__ addend_hi,
                                                          uint64_t addend_bs, uint32_t comp0, uint32_t n_comps, uint32_t galois) {
    constexpr uint32_t N = 256u << LOG_R;
    __shared__ double lds[4 * kRowPitch];
    const uint32_t rg = blockIdx.x, i = blockIdx.y;
    // batch items in descending order: the conversion kernel before this one wrote them in ascending order, so the most
    // recently written ones, still in the last-level cache, are read first (4-5 % on this kernel in batched calls)
    const uint32_t zz = gridDim.z - 1 - blockIdx.z;
    const uint32_t b = zz / n_comps, comp = comp0 + (zz - b * n_comps);
    const void* adp = nullptr;
    const uint8_t* adp_hi = nullptr;
    double admul = 0.0;
    if constexpr (ADDEND != 0) {
        const uint64_t ad_off = (uint64_t)b * addend_bs + ((uint64_t)comp * ell + i) * N;
        if constexpr (ADF == 1) {
            adp = static_cast<const uint32_t*>(addend) + ad_off;
            adp_hi = addend_hi + ad_off;
        } else if constexpr (ADF == 2) {
            adp = static_cast<const uint32_t*>(addend) + ad_off;
        } else {
            adp = static_cast<const uint64_t*>(addend) + ad_off;
        }
    }
    if constexpr (ADDEND == 2) admul = addend_mul[i];
    const uint64_t conv_off = (((uint64_t)b * 2 + comp) * ell + i) * N;
    const void* ap;
    const uint8_t* ap_hi = nullptr;
    if constexpr (ACCP) {
        ap = static_cast<const uint32_t*>(acc) + conv_off;
        ap_hi = acc_hi + conv_off;
    } else {
        ap = static_cast<const uint64_t*>(acc) + (((uint64_t)b * 2 + comp) * E + i) * N;
    }
    task_rows_finish<LOG_R, GATHER, ADDEND, W, ACCP, ADF>(tw, mods[i], i, Pinv[i], admul, conv + conv_off, ap, ap_hi,
                                                          out + (uint64_t)b * out_bs + ((uint64_t)comp * out_limbs + i) * N, adp,
                                                          adp_hi, galois, rg, threadIdx.x, lds);
}

void launch_rows_moddown_finish(const ks_ctx* c, const Level& lv, const uint64_t* acc, const uint64_t* conv, void* out_words,
                                uint64_t out_bs, const void* addend, uint64_t addend_bs, uint32_t addend_comps,
                                uint32_t galois, uint32_t batch, hipStream_t s, const FinishScale* fs, bool out_words32,
                                const PackedDigits* acc_packed, const PackedDigits* addend_packed) {
    if (batch == 0) return;
    const void* addend_p = addend_packed ? static_cast<const void*>(addend_packed->lo) : addend;
    const uint8_t* addend_h = addend_packed ? addend_packed->hi : nullptr;
    const double* mul = fs ? fs->mul : c->d_Pinv;
    const double* admul = fs ? fs->addend_mul : nullptr;
    const uint32_t out_limbs = fs ? fs->out_limbs : lv.ell;
    if (out_limbs == 0) return;
    if (!addend_p) addend_comps = 0;
    ProfScope ps("rows_moddown_finish",
                 (double)batch * out_limbs *
                     (2 * 8 + 2 * (acc_packed ? 5 : 8) + (out_words32 ? 1 : 2) * 8 + addend_comps * (addend_packed ? 5 : out_words32 ? 4 : 8)) * c->N,
                 s);
    const dim3 block(64);
    const uint32_t row_groups = c->N / 1024;
    const void* accp = acc_packed ? static_cast<const void*>(acc_packed->lo) : static_cast<const void*>(acc);
    const uint8_t* acch = acc_packed ? acc_packed->hi : nullptr;
    // one launch for the components that take the addend, one for those that do not
    for (int pass = 0; pass < 2; ++pass) {
        const uint32_t comp0 = pass == 0 ? 0 : addend_comps, n_comps = pass == 0 ? addend_comps : 2 - addend_comps;
        if (n_comps == 0) continue;
        const int mode = pass == 1 ? 0 : (admul ? 2 : 1);
        const dim3 grid(row_groups, out_limbs, batch * n_comps);
#define KS_LAUNCH_FINISH_P(LOGR, GATHER, MODE, WT, ACCP, ADF)                                                                      \
    hipLaunchKernelGGL((rows_moddown_finish<LOGR, GATHER, MODE, WT, ACCP, ADF>), grid, block, 0, s, c->tw_fwd, c->d_mod, mul, admul, \
                       lv.ell, lv.E, out_limbs, accp, acch, conv, static_cast<WT*>(out_words), out_bs, addend_p, addend_h, addend_bs, \
                       comp0, n_comps, galois)
    // Who calls: a scaled addend is packed and comes with a packed accumulator (multiplications); an addend as it is comes with
    // a packed accumulator, in the word size of the output (hoisted rotations).
#define KS_LAUNCH_MODES(LOGR, WT, ADF)                                                  \
    if (mode == 2) KS_LAUNCH_FINISH_P(LOGR, false, 2, WT, true, 1);                     \
    else if (mode == 1 && galois != 1) KS_LAUNCH_FINISH_P(LOGR, true, 1, WT, true, ADF);  \
    else if (mode == 1) KS_LAUNCH_FINISH_P(LOGR, false, 1, WT, true, ADF);              \
    else if (acc_packed) KS_LAUNCH_FINISH_P(LOGR, false, 0, WT, true, 0);               \
    else KS_LAUNCH_FINISH_P(LOGR, false, 0, WT, false, 0)
#define KS_LAUNCH(LOGR)                                      \
    if (out_words32) { KS_LAUNCH_MODES(LOGR, uint32_t, 2); } \
    else { KS_LAUNCH_MODES(LOGR, uint64_t, 0); }
        KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_MODES
#undef KS_LAUNCH_FINISH_P
    }
}

// ------------------------------------------------------------------------------------------------
// Rescale.  The rescale's remainder r = (sum - conv)[ell-1] P^-1 (coefficient domain, centred) has to be subtracted from every
// other limb after the division by P: (acc_i - conv_i) P^-1 + d_i - r, times q_{ell-1}^-1.  As P r joins conv_i before the
// forward transform, it costs one more source of that conversion, and the rescale needs no transforms of its own (a
// forward transform and two more passes over every limb: 290 of 1310 us per 8 multiplications at L = 35).
// With y_k = [x_k (P / p_k)^-1]_{p_k} the converted special part of limb ell-1 times P^-1 is sum_k y_k p_k^-1.
// One thread per coefficient, K + 1 limbs read and one written.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rescale_remainder_kernel(Mod m, const double* __restrict__ pinv, uint32_t ell, uint32_t K,
                                                                uint32_t N, uint64_t* __restrict__ acc) {
    const uint32_t n = blockIdx.x * 256 + threadIdx.x;
    uint64_t* last = acc + ((uint64_t)blockIdx.y * (ell + K) + ell - 1) * N + n;
    static_assert(kMaxLimbsIn <= kMacTerms, "products per exact sum");
    double hi = kMacBias, lo = 0.0;
#pragma unroll 4
    for (uint32_t k = 0; k < K; ++k) mac_exact(load_f64(last + (uint64_t)(k + 1) * N), pinv[k], hi, lo);
    const double r = canon(reduce_lazy(load_f64(last) - mac_reduce(hi, lo, m), m), m);
    store_f64(last, r > (m.p - 1.0) * 0.5 ? r - m.p : r);
}

void launch_rescale_remainder(const ks_ctx* c, const Level& lv, uint64_t* acc, uint32_t n_polys, hipStream_t s) {
    if (n_polys == 0) return;
    ProfScope ps("rescale_remainder", (double)n_polys * (c->K + 2) * c->N * 8.0, s);
    const uint64_t q = c->mod[lv.ell - 1];
    hipLaunchKernelGGL(rescale_remainder_kernel, dim3(c->N / 256, n_polys), dim3(256), 0, s, Mod{(double)q, 1.0 / (double)q}, lv.d_pinv_last,
                       lv.ell, c->K, c->N, acc);
}

}  // namespace ks
