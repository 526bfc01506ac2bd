// Vertically fused kernels of the key-switching chain (the paper's vertical fusion: dependent limb
// operations on the same positions stay in registers instead of making a round trip through memory).
//
//  * bconv_ntt_cols       base conversion of a digit feeding the column half of the forward transform of
//                         each target limb: the converted limb never exists in memory in coefficient form.
//  * rows_inner_product   row half of the forward transform of every raised limb feeding the inner product
//                         with the key: the raised limb never exists in memory in evaluation form.  In calls of several
//                         ciphertexts the ciphertext limbs' sums meet the converted limbs there and do not exist in memory either.
//  * rows_moddown_finish  row half of the forward transform of the converted special part feeding
//                         (acc - conv) * P^-1 (+ addend).
//
// Base conversion is coefficient-wise and the column half touches a fixed set of coefficient positions per
// tile, so the first fusion is legal; the inner product and the final scale are slot-wise and the row half
// produces complete slots, so the other two are.
#include "ks_internal.hpp"
#include "ks_tasks.hpp"

namespace ks {

// The 16 positions of a source that a thread owns, as they lie in memory (kDigitBias).
struct SourceRaw {
    Words4 lo[4], top;
};
template <int LOG_R>
__device__ __forceinline__ SourceRaw load_source(BufferRsrc rsrc, uint32_t limb, uint32_t lo_off, uint32_t top_off) {
    constexpr uint32_t N = 256u << LOG_R;
    const uint32_t base = limb * (uint32_t)packed_limb_bytes(N);
    SourceRaw r;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        r.lo[q] = __builtin_bit_cast(Words4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)lo_off, (int)(base + q * 4096), 0));
    r.top = __builtin_bit_cast(Words4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)top_off, (int)(base + 4 * N), 0));
    return r;
}

// One source of a conversion: acc[t][k] += (y[k] + 0x80808080) * f[t] as exact integers (the constant is taken out by what acc
// starts from).  The 40 bits of a source point are cut once into PIECES whole numbers, every target adds PIECES products
// against its centred factors; the bounds of these sums are stated at cut_source.
template <int TS, int PIECES>
__device__ __forceinline__ void bconv_accumulate(double (&acc)[TS][16], const SourceRaw& y, const double (&f)[TS][3]) {
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint32_t w = y.lo[k >> 2].w[k & 3];
        const int top = (int)(y.top.w[k >> 2] << (24 - 8 * (k & 3))) >> 24;
        double p[PIECES];
        cut_source<PIECES>(w, top, p);
#pragma unroll
        for (int tt = 0; tt < TS; ++tt)
#pragma unroll
            for (int i = 0; i < PIECES; ++i) acc[tt][k] = __builtin_fma(p[i], f[tt][i], acc[tt][k]);
    }
}

// ------------------------------------------------------------------------------------------------
// y: [poly][..] packed sources y_i = [x_i N^-1 (D/s_i)^-1]_{s_i} (written by inv_cols_packed with its scale table).  Each
// workgroup owns one column tile (4096 positions) and TS targets of one digit: it accumulates sum_i y_i * (D/s_i mod t) as
// an exact integer for its 16 positions per thread, then runs the column stages of the forward transform modulo t and stores
// packed limbs.  The sources are re-read by the workgroups of the other target subsets; those reads are served by L2 / the
// last-level cache.
// ------------------------------------------------------------------------------------------------
// PIECES: 3 in general (moduli below 2^36); 2 when every modulus of the context is below 2^32 (the plan's factors are
// then cut at 16 bits: two products per source and target instead of three).
template <int LOG_R, int TS, int PIECES>
__global__ __launch_bounds__(256) void bconv_ntt_cols(const double* __restrict__ tw, const BConvPlan* __restrict__ plans,
                                                      const uint8_t* __restrict__ y, uint64_t y_ps, uint8_t* __restrict__ out,
                                                      uint64_t out_ps, uint32_t n_subsets) {
    constexpr uint32_t N = 256u << LOG_R, TILES = 1u << (LOG_R - 4), TC = 256 / TILES;
    __shared__ double lds[LOG_R > 4 ? 4096 : 1];
    const uint32_t tid = threadIdx.x, tile = blockIdx.x;
    const uint32_t plan_id = blockIdx.y / n_subsets, subset = blockIdx.y - plan_id * n_subsets;
    const BConvPlan& P = plans[plan_id];
    const int n_dst = (int)P.n_dst, n_src = (int)P.n_src;
    const int t0 = (int)subset * TS;
    if (t0 >= n_dst) return;  // uniform for the whole workgroup
    const uint8_t* yp = y + (uint64_t)blockIdx.z * y_ps;
    uint8_t* op = out + (uint64_t)blockIdx.z * out_ps;
    const uint32_t c = tid & (TC - 1), r0 = tid / TC, col = tile * TC + c;

    // Per-target constants.  They are uniform across the workgroup and travel through scalar loads.
    Mod mt[TS];
    const double* hat_row[TS];
    double acc[TS][16];
#pragma unroll
    for (int tt = 0; tt < TS; ++tt) {
        const int t = min(t0 + tt, n_dst - 1);  // a ragged last subset recomputes its last target (stored once)
        mt[tt] = P.dst_mod[t];
        hat_row[tt] = &P.hats[t][0][0];
        const double start = P.dst_start[t];
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[tt][k] = start;
    }

    // Software pipeline over the sources, two per trip so that the points and the uniform factors can alternate between two
    // register sets, with the limb index of the source after next fetched ahead as well: nothing is waited for right after it was
    // requested.  Sources past the end are zero-padded in the plan (factor 0, a valid limb): prefetches are unconditional -- a
    // conditional one would make the wait-count bookkeeping assume the worst at the join and stall every use on the
    // newest loads -- and an odd source count simply runs one padding source.  The factors of the next source are requested
    // before the products of the current one: scalar loads complete out of order, so the first use of f waits for every
    // scalar load in flight, and at that moment only f's own, requested a source ago, should be.  The points are read through
    // a buffer descriptor of this polynomial's bundle: per-lane offset in a vector register, limb and row offset in a
    // scalar one, so switching limb costs no vector instructions.
    const BufferRsrc ysrd = make_buffer_rsrc(yp, y_ps);
    const uint32_t lo_off = (r0 * 1024 + col) * 16, top_off = source_bytes_offset(r0, col);
    const auto load_factors = [&](double (&f)[TS][3], int i) {
#pragma unroll
        for (int tt = 0; tt < TS; ++tt)
#pragma unroll
            for (int p = 0; p < PIECES; ++p) f[tt][p] = hat_row[tt][i * 4 + (p + 1 < PIECES ? p : 3)];
    };
    SourceRaw ya = load_source<LOG_R>(ysrd, P.src_limb[0], lo_off, top_off), yb;
    double fa[TS][3], fb[TS][3];
    load_factors(fa, 0);
    uint32_t limb_next = P.src_limb[1];
#pragma unroll 1
    for (int i = 0; i < n_src; i += 2) {
        yb = load_source<LOG_R>(ysrd, limb_next, lo_off, top_off);
        load_factors(fb, min(i + 1, kMaxSrc - 1));
        limb_next = P.src_limb[min(i + 2, kMaxSrc - 1)];
        __builtin_amdgcn_sched_barrier(0);
        bconv_accumulate<TS, PIECES>(acc, ya, fa);
        __builtin_amdgcn_sched_barrier(0);
        ya = load_source<LOG_R>(ysrd, limb_next, lo_off, top_off);
        load_factors(fa, min(i + 2, kMaxSrc - 1));
        limb_next = P.src_limb[min(i + 3, kMaxSrc - 1)];
        __builtin_amdgcn_sched_barrier(0);
        bconv_accumulate<TS, PIECES>(acc, yb, fb);
        __builtin_amdgcn_sched_barrier(0);
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
            packed_store<256>(op + (uint64_t)P.dst_limb[t] * packed_limb_bytes(N), N, r0 * 1024 + col, pack(acc[tt]));
            if constexpr (LOG_R > 4) __syncthreads();  // the exchange buffer is reused by the next target
        }
    }
}

// Which kernel the two conversions of a call take: 0 vector, 8 or 16 matrix cores with tiles of 8 or 16 columns.  One answer
// for both: the code of a kernel that ran a moment ago is still in the caches, so a call that mixes them pays 1-2 us at
// small sizes and 5-8 where its data exceed the memory-side cache.
//   G counts the matrix-core kernel's workgroups at six targets and 2048 positions each.  Their cost hardly depends on the sources; the
// vector kernel takes one instruction per source and piece of a residue (three pieces, two for moduli below 2^32) and some for the
// transform.  So the line is drawn by the load, the vector instructions that a group of six targets replaces, 20 per target besides
// the products: many sources and full groups (20 targets take four, 24 too) favour the matrix cores.  Checked on 1786 key-switches of
// random shapes (N = 2^12 .. 2^16, one to eight ciphertexts, both word sizes), each with every kernel and number of targets: the choice
// is within 0.1 % (N = 2^12) to 1.5 % (2^14) of the best one on average.  Matrix cores with one target a lane half against the vector
// kernel with its number of targets, by load per group, 36-bit moduli, N = 2^16, launches of 1024 to 4096 vector workgroups of one target:
// below 130 +1.8 %, 130-160 -0.6, 160-200 -1.9, above 200 -5.1; 28-bit +3.5, +1.8, -0.3, -1.0; N = 2^15, 256 to 512 workgroups: 36-bit
// 0.0, -1.3, -3.6, -5.7; 28-bit +1.9, +0.1, -2.2, -3.5.  Where a launch has just more than 256 or 512 groups a few compute units do twice
// the work of the others, hence the extra.
//   16 columns are whole lines, but one workgroup of 512 threads per compute unit that works in step: ahead when a launch
// has six rounds or more, full groups and (28-bit moduli) four thousand groups.
//   Below N = 2^15 launches are at their floor; the vector kernel with one target per workgroup and the matrix cores are within 2 %.
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

void launch_bconv_ntt_cols(const ks_ctx* c, const PlanSet& plans, uint32_t limbs_moved_per_poly, const uint8_t* y, uint64_t y_ps,
                           uint8_t* out, uint64_t out_ps, uint32_t n_polys, int tile, hipStream_t s) {
    const uint32_t n_plans = plans.n_plans, max_targets = plans.max_targets;
    const BConvPlan* d_plans = plans.d_plans;
    if (n_polys == 0 || n_plans == 0) return;
    const int kernel = c->opt[KS_OPT_BCONV_KERNEL] ? c->opt[KS_OPT_BCONV_KERNEL] : (tile ? 2 : 1);
    if (kernel == 2) {
        // algorithmic vector work per coefficient and target of this kernel: 9 to recombine and reduce the five sums, 4 a column stage, 3 to
        // pack (the sources come cut into bytes; the contraction runs on the matrix cores: 25 int8 multiply-adds per source and target)
        const double vec_ops = plans.targets * (12.0 + 4.0 * (c->logN - 8));
        ProfScope ps("bconv_mfma_ntt_cols", (double)limbs_moved_per_poly * n_polys * packed_limb_bytes(c->N), s, vec_ops * n_polys * c->N);
        // Targets per lane half.  A workgroup with one needs half the registers and a third of the time, so that four share a compute unit
        // and a launch of a few rounds ends evenly: one key-switch 8 -> 24 93.0 -> 90.2 us, one merged multiplication 104.7 -> 100.3,
        // ten of 4 -> 12 at N = 2^15 -6 %.  Three read the sources once for three: ahead for whole-line tiles (hoisted rotations 9935 ->
        // 9641 us, 64 multiplications 7083 -> 6984) and where sources are many and the launch is not small (15 -> 17 x 4, 255 -> 232).
        const uint64_t sixes = (uint64_t)(c->N / 2048) * plans.sixes * n_polys;
        const int tl = c->opt[KS_OPT_BCONV_TARGETS] ? (c->opt[KS_OPT_BCONV_TARGETS] == 3 ? 3 : 1)
                       : tile == 16 || (mfma_sources(plans.shape_src) >= 8 && sixes >= 384) ? 3 : 1;
        launch_bconv_mfma_ntt_cols(c, plans, y, y_ps, out, out_ps, n_polys, tl, tile == 16, s);
        return;
    }
    // Targets per workgroup; the context option KS_OPT_BCONV_TARGETS overrides the choice.
    const uint32_t tiles = 1u << (c->logN - 12);
    const int ts = c->opt[KS_OPT_BCONV_TARGETS] ? c->opt[KS_OPT_BCONV_TARGETS] : vector_conversion_targets(plans, tiles, n_polys);
    const uint32_t n_subsets = (max_targets + ts - 1) / ts;
    const dim3 grid(tiles, n_plans * n_subsets, n_polys), block(256);
    // algorithmic fp64 work per coefficient: an FMA per source, target and piece, then per target one reduction and the column stages
    // (8 per butterfly, half a butterfly per point and stage)
    const double ops = (double)c->pieces * plans.products + plans.targets * (3.0 + 4.0 * (c->logN - 8));
    ProfScope ps("bconv_ntt_cols", (double)limbs_moved_per_poly * n_polys * packed_limb_bytes(c->N), s, ops * n_polys * c->N);
#define KS_LAUNCH_BCONV(LOGR, TSV)                                                                                                      \
    if (c->pieces == 2)                                                                                                                 \
        hipLaunchKernelGGL((bconv_ntt_cols<LOGR, TSV, 2>), grid, block, 0, s, c->d_tw_fwd, d_plans, y, y_ps, out, out_ps,  \
                           n_subsets);                                                                                                  \
    else                                                                                                                                \
        hipLaunchKernelGGL((bconv_ntt_cols<LOGR, TSV, 3>), grid, block, 0, s, c->d_tw_fwd, d_plans, y, y_ps, out, out_ps,  \
                           n_subsets)
#define KS_LAUNCH(LOGR)                             \
    if (ts == 4) { KS_LAUNCH_BCONV(LOGR, 4); }      \
    else if (ts == 3) { KS_LAUNCH_BCONV(LOGR, 3); } \
    else if (ts == 2) { KS_LAUNCH_BCONV(LOGR, 2); } \
    else { KS_LAUNCH_BCONV(LOGR, 1); }
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_BCONV
}

// Digits that rows_split takes: its LDS stays below 64 KB.
constexpr uint32_t kSplitDigits = 4;
static_assert(rows_split_lds(kSplitDigits) <= 65536, "LDS of rows_split");

// Where the sums of a launch go (SumsEnd of every batch item).
template <typename W>
struct SumsOut {
    uint8_t* acc;               // [b][2][E] packed
    const uint8_t* addend;      // [b][2][ell] packed, or null (FINISH == 0: of the limb that is dropped)
    double drop_mul;
    const uint8_t* conv;        // [b][2][ell] packed
    W* out;                     // [b][2][n_pos] words, batch items out_bs apart
    uint64_t out_bs;
    const double *mul, *addend_mul;   // by limb
};
template <int FINISH, typename W>
__device__ __forceinline__ SumsEnd<W> sums_end(const SumsOut<W>& o, uint32_t b, uint32_t pos, uint32_t ell, uint32_t E, uint32_t n_pos, uint32_t N) {
    const uint64_t limb = packed_limb_bytes(N);
    SumsEnd<W> end{};
    if constexpr (FINISH == 0) {
        end.acc = o.acc + (uint64_t)b * 2 * E * limb;
        end.drop = o.addend ? o.addend + (uint64_t)b * 2 * ell * limb : nullptr;
        end.drop_mul = o.drop_mul;
    } else {
        end.conv = o.conv + (uint64_t)b * 2 * ell * limb;
        if constexpr (FINISH == 2) end.addend = o.addend + (uint64_t)b * 2 * ell * limb;
        end.out = o.out + (uint64_t)b * o.out_bs + (uint64_t)pos * N;
        end.out_comp = (uint64_t)n_pos * N;
        end.mul = o.mul[pos];
        if constexpr (FINISH == 2) end.admul = o.addend_mul[pos];
    }
    return end;
}

// ------------------------------------------------------------------------------------------------
// Inner product with the key: sum[c][pos] = sum_j d~_j[pos] * key[j][c][m(pos)].  For pos inside digit j, d~_j[pos] is the input limb
// itself; otherwise it is the raised limb, whose row half of the forward transform is done here.
// A workgroup = four rows of one limb position; it walks the digits, so d~ is read once and feeds both key
// components (load reuse).
//   Calls of several ciphertexts run it twice (sums_meet_division): ahead of the division on the limbs that the division drops (FINISH == 0),
// and as its last kernel on the limbs that stay (FINISH > 0), where the sums meet the converted limbs in registers and never exist
// in memory.
// ------------------------------------------------------------------------------------------------
// WD / WK: word types of d (uint8_t: packed) and of the key; the output has the key's.
template <int LOG_R, typename WD, typename WK, bool PREFETCH, int FINISH>
__global__ __launch_bounds__(64, 2) void rows_inner_product(TwTables tw, TwTables twi, const Mod* __restrict__ mods, DigitRanges dg,
                                                         uint32_t ell, uint32_t E, uint32_t L, uint32_t M,
                                                         const WD* __restrict__ d, uint64_t d_ps,
                                                         const uint8_t* __restrict__ lifted, const WK* __restrict__ evk,
                                                         SumsOut<WK> o, uint32_t pos0, uint32_t n_pos, uint32_t batch, uint32_t special_first) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R;
    constexpr uint64_t LIMB = packed_limb_bytes(N);
    __shared__ InnerProductLds lds;
    // Workgroup -> (row group, limb position, batch item).  Consecutive workgroup ids go to the eight XCDs in
    // turn, each with its own L2; the ids that land on one XCD walk through all batch items of one
    // (row group, position) tile before moving to the next tile, so the key slots and twiddles of a tile are
    // fetched into that L2 once and reused by the whole batch.
    const uint32_t slot = blockIdx.x >> 3, b = slot % batch, tile = (slot / batch) * 8 + (blockIdx.x & 7);
    if (tile >= (R / 4) * n_pos) return;  // uniform: padding workgroups when the tile count is not a multiple of 8
    // special_first (launches whose wavefronts are all resident at once, i.e. a single ciphertext): the special limbs take
    // the first workgroup ids.  Their wavefronts have the most arithmetic after their last load (one more transform and the
    // two inverse row passes) and the memory system serves the earliest requests first, so started last they are the tail
    // of the launch (59 k cycles per special wavefront against 37 k for the others; 40.2 -> 37.1 us per launch).  Batched
    // launches keep them last: the next kernel reads exactly these limbs and finds them cached (0.5-2 % per call).
    const uint32_t rg = tile % (R / 4), slot_pos = tile / (R / 4), n_special = E - ell;
    const uint32_t pos = !special_first ? pos0 + slot_pos : slot_pos < n_special ? ell + slot_pos : slot_pos - n_special;
    task_rows_inner_product<LOG_R, WD, WK, PREFETCH, FINISH>(tw, twi, mods, dg, ell, E, L, M, d + (uint64_t)b * d_ps,
                                                             lifted + (uint64_t)b * dg.ndig * E * LIMB, evk,
                                                             sums_end<FINISH>(o, b, pos, ell, E, n_pos, N), pos, rg, threadIdx.x, lds);
}

template <int LOG_R, typename WD, typename WK>
__global__ __launch_bounds__(64 * (kSplitDigits + 2), 2) void rows_inner_product_split(TwTables tw, TwTables twi, const Mod* __restrict__ mods,
                                                      DigitRanges dg, uint32_t ell, uint32_t E, uint32_t L, uint32_t M,
                                                      const WD* __restrict__ d, uint64_t d_ps, const uint8_t* __restrict__ lifted,
                                                      const WK* __restrict__ evk, uint8_t* __restrict__ acc,
                                                      const uint8_t* __restrict__ drop, double drop_mul, uint32_t batch) {
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R;
    constexpr uint64_t LIMB = packed_limb_bytes(N);
    extern __shared__ double split_lds[];
    const uint32_t slot = blockIdx.x >> 3, b = slot % batch, tile = (slot / batch) * 8 + (blockIdx.x & 7);   // as above
    if (tile >= (R / 4) * E) return;  // uniform
    const uint32_t rg = tile % (R / 4), slot_pos = tile / (R / 4), n_special = E - ell, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t pos = slot_pos < n_special ? ell + slot_pos : slot_pos - n_special;   // the longest chains first
    SumsEnd<WK> end{};
    end.acc = acc + (uint64_t)b * 2 * E * LIMB;
    end.drop = drop ? drop + (uint64_t)b * 2 * ell * LIMB : nullptr;
    end.drop_mul = drop_mul;
    task_rows_split<LOG_R, WD, WK>(tw, twi, mods, dg, ell, E, L, M, d + (uint64_t)b * d_ps, lifted + (uint64_t)b * dg.ndig * E * LIMB, evk,
                                   end, pos, rg, wave, threadIdx.x & 63u, split_lds);
}

// Workgroups of a launch over n_pos limb positions.
static uint32_t sums_grid(const ks_ctx* c, uint32_t n_pos, uint32_t batch) { return (c->N / 1024 * n_pos + 7) / 8 * 8 * batch; }

// Sums that meet the division save 10 bytes of traffic a residue of the ciphertext limbs, a seventh of a key-switch's; but two launches, the
// first of them over the limbs that the division drops alone, need work for the whole chip each.  The line is at three and a half wavefronts per
// SIMD in a launch over all limbs.  Calls (N = 2^14: in several passes) in two launches against one and a kernel of its own for the division, us,
// by wavefronts of that launch: N = 2^16, 24 limbs, 2048 102.5 / 98.4, 4096 148.7 / 149.5, 6144 198.3 / 206.4, 8192 243.5 / 258.0, 12288
// 345.2 / 368.1; 28 bits 4096 133.7 / 135.8, 8192 214.5 / 226.6; 21 limbs multiplied 3712 179.1 / 177.8, 7424 288.6 / 294.5, 14848 536 / 563;
// N = 2^15 2048 96.2 / 88.5, 4096 140.7 / 140.6, 8192 232.4 / 247.1; N = 2^14 2048 92.1 / 84.3, 3840 293.8 / 302.7.
//   More than four digits make the traffic saved a smaller part and a wavefront, and so the last round, longer: five, 3840 152.2 / 147.2 and
// 170.3 / 167.4, 6144 248.2 / 251.1; six, 4480 205.0 / 210.7; seven, 3680 204.7 / 198.2; eight, 9216 466.5 / 473.0.
//   And a launch of the limbs that stay for itself: 512 wavefronts of 4096 83.9 / 80.0, 832 of 6656 120.1 / 116.6, 1280 of 4864 101.7 / 98.9 and of
// 4160 91.6 / 92.4, 1536 of 5632 111.9 / 113.2, 1664 of 8320 141.2 / 142.9; multiplications 256 of 4096 91.9 / 87.6, 1152 of 4032 114.0 / 112.1,
// 1536 of 6656 146.6 / 148.5.
bool sums_meet_division(const ks_ctx* c, const Level& lv, uint32_t n_stay, uint32_t batch) {
    return sums_grid(c, lv.E, batch) > (lv.ndig > 4 ? 4096 : 3584) && sums_grid(c, n_stay, batch) > 1280;
}

// A wavefront per digit and component where all workgroups are resident at once, three a compute unit (118 registers and 42 KB of LDS at
// three digits) or two (four digits); fewer digits have less to take apart.  One key-switch, a wavefront for everything -> split: three
// digits, N = 2^12, 256 workgroups 39.1 -> 33.1 us, N = 2^14 512 48.6 -> 44.1, 768 54.6 -> 53.5, but 1024 59.8 -> 64.8; N = 2^15 256
// 49.0 -> 45.0, 800 59.7 -> 63.9; four, N = 2^13 384 45.3 -> 37.8; two, N = 2^12 48 33.6 -> 29.8, N = 2^13 192 38.0 -> 34.5, N = 2^15 576
// 52.0 -> 53.3; one, N = 2^12 128 33.2 -> 31.4, N = 2^14 512 41.2 -> 42.1.
static bool split_sums(const ks_ctx* c, const Level& lv, uint32_t batch) {
    constexpr uint32_t most[kSplitDigits] = {256, 512, 768, 512};
    return lv.ndig <= kSplitDigits && sums_grid(c, lv.E, batch) <= most[lv.ndig - 1];
}

template <int FINISH, typename WK>
static void launch_rows_sums(const ks_ctx* c, const Level& lv, const void* d, uint64_t d_ps, const uint8_t* lifted, const void* evk,
                             const SumsOut<WK>& o, uint32_t pos0, uint32_t n_pos, uint32_t batch, hipStream_t s, int d_word) {
    DigitRanges dg;
    dg.ndig = lv.ndig;
    for (uint32_t j = 0; j < kMaxDigits; ++j) {
        dg.lo[j] = j < lv.ndig ? lv.digit_lo[j] : 0;
        dg.hi[j] = j < lv.ndig ? lv.digit_hi[j] : 0;
    }
    const uint32_t grid = sums_grid(c, n_pos, batch);
    // launches with more than two wavefronts per SIMD (1024 SIMDs) to run take the variant that requests the next digit's
    // loads early (3 % faster there); the single-ciphertext launch is bound by
    // bandwidth and gains nothing from it
    const bool prefetch = grid > 2048, all = FINISH == 0 && n_pos == lv.E;
    const bool split = all && split_sums(c, lv, batch);
#define KS_LAUNCH_IP(LOGR, WDT, PF)                                                                                                            \
    hipLaunchKernelGGL((rows_inner_product<LOGR, WDT, WK, PF, FINISH>), dim3(grid), dim3(64), 0, s, c->tw_fwd, c->tw_inv, c->d_mod, dg, lv.ell, \
                       lv.E, c->L, c->M, static_cast<const WDT*>(d), d_ps, lifted, static_cast<const WK*>(evk), o, pos0, n_pos, batch,          \
                       all && !prefetch ? 1u : 0u)
#define KS_LAUNCH_SPLIT(LOGR, WDT)                                                                                                             \
    hipLaunchKernelGGL((rows_inner_product_split<LOGR, WDT, WK>), dim3(grid), dim3(64 * (lv.ndig + 2)), rows_split_lds(lv.ndig), s, c->tw_fwd,  \
                       c->tw_inv, c->d_mod, dg, lv.ell, lv.E, c->L, c->M, static_cast<const WDT*>(d), d_ps, lifted,                            \
                       static_cast<const WK*>(evk), o.acc, o.addend, o.drop_mul, batch)
#define KS_LAUNCH_WD(LOGR, WDT)                           \
    if (split) KS_LAUNCH_SPLIT(LOGR, WDT);                \
    else if (prefetch) KS_LAUNCH_IP(LOGR, WDT, true);     \
    else KS_LAUNCH_IP(LOGR, WDT, false)
#define KS_LAUNCH(LOGR)                                                     \
    if constexpr (FINISH == 1) { KS_LAUNCH_IP(LOGR, WK, true); }            \
    else if constexpr (FINISH == 2) { KS_LAUNCH_IP(LOGR, uint8_t, true); }  \
    else if (d_word == 1) { KS_LAUNCH_WD(LOGR, uint8_t); }                  \
    else { KS_LAUNCH_WD(LOGR, WK); }
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_WD
#undef KS_LAUNCH_SPLIT
#undef KS_LAUNCH_IP
}

// bytes that a launch over n_pos positions, `own` of them in a digit of their own, reads of d, the raised limbs and the key (once per call)
static double sums_bytes(const Level& lv, uint32_t n_pos, uint32_t own, uint32_t batch, int d_word, bool words32) {
    return (double)batch * (5.0 * (lv.ndig * n_pos - own) + (d_word == 1 ? 5.0 : d_word) * own) + (words32 ? 4.0 : 8.0) * 2.0 * lv.ndig * n_pos;
}

void launch_rows_inner_product(const ks_ctx* c, const Level& lv, const void* d, uint64_t d_ps, const uint8_t* lifted,
                               const void* evk, uint8_t* acc, uint32_t batch, hipStream_t s, int d_word, bool words32,
                               const uint8_t* drop_addend, bool dropped_only) {
    if (batch == 0) return;
    const uint32_t pos0 = !dropped_only ? 0 : drop_addend ? lv.ell - 1 : lv.ell, n_pos = lv.E - pos0;
    ProfScope ps(!dropped_only && split_sums(c, lv, batch) ? "rows_inner_product_split" : "rows_inner_product",
                 (sums_bytes(lv, n_pos, lv.ell - pos0, batch, d_word, words32) + 10.0 * batch * n_pos) * c->N, s);
    const auto launch = [&](auto word) {
        using WK = decltype(word);
        SumsOut<WK> o{};
        o.acc = acc;
        o.addend = drop_addend;
        o.drop_mul = lv.Pmod_last;
        launch_rows_sums<0, WK>(c, lv, d, d_ps, lifted, evk, o, pos0, n_pos, batch, s, d_word);
    };
    if (words32) launch(uint32_t{});
    else launch(uint64_t{});
}

void launch_rows_key_finish(const ks_ctx* c, const Level& lv, const void* d, uint64_t d_ps, const uint8_t* lifted, const void* evk,
                            const uint8_t* conv, const uint8_t* addend, void* out, uint64_t out_bs, uint32_t batch, hipStream_t s,
                            int d_word, bool words32, const FinishScale* fs) {
    const uint32_t n_pos = fs ? fs->out_limbs : lv.ell;
    if (batch == 0 || n_pos == 0) return;
    ProfScope ps("rows_key_finish",
                 (sums_bytes(lv, n_pos, n_pos, batch, d_word, words32) + (double)batch * n_pos * (10.0 + (fs ? 10.0 : 0.0) + (words32 ? 8.0 : 16.0))) * c->N, s);
    const auto launch = [&](auto word) {
        using WK = decltype(word);
        SumsOut<WK> o{};
        o.conv = conv;
        o.addend = addend;
        o.out = static_cast<WK*>(out);
        o.out_bs = out_bs;
        o.mul = fs ? fs->mul : c->d_Pinv;
        o.addend_mul = fs ? fs->addend_mul : nullptr;
        if (fs) launch_rows_sums<2, WK>(c, lv, d, d_ps, lifted, evk, o, 0, n_pos, batch, s, d_word);
        else launch_rows_sums<1, WK>(c, lv, d, d_ps, lifted, evk, o, 0, n_pos, batch, s, d_word);
    };
    if (words32) launch(uint32_t{});
    else launch(uint64_t{});
}

// ------------------------------------------------------------------------------------------------
// out[b][comp][i] = (acc[b][comp][i] - NTT_rows(conv[b][comp][i])) * P^-1 (+ addend), canonical.
// ------------------------------------------------------------------------------------------------
// ADDEND: 0 = none, 1 = words of component 0, read through sigma_galois and added as they are, 2 = packed ([b][2][ell]), multiplied by
// addend_mul[i] first.  Compile-time so that the kernel has no branch in front of its loads; the components that take no addend
// in mode 1 branch to the other instance of the task, which is uniform.
// A launch covers n_rot rotations (1 but for hoisted ones) of every batch item: acc [rot][b][2][E], conv [rot][b][2][ell].
template <int LOG_R, int ADDEND, typename W>
__global__ __launch_bounds__(64) void rows_moddown_finish(TwTables tw, const Mod* __restrict__ mods,
                                                          const double* __restrict__ Pinv, const double* __restrict__ addend_mul,
                                                          uint32_t ell, uint32_t E, uint32_t out_limbs, const uint8_t* __restrict__ acc,
                                                          const uint8_t* __restrict__ conv, W* __restrict__ out, uint64_t out_bs, uint64_t out_rs,
                                                          const void* __restrict__ addend, uint64_t addend_bs, uint32_t batch, FinishRotations rot) {
    constexpr uint32_t N = 256u << LOG_R;
    constexpr uint64_t LIMB = packed_limb_bytes(N);
    __shared__ double lds[4 * kRowPitch];
    const uint32_t rg = blockIdx.x, i = blockIdx.y;
    // batch items in descending order: the conversion kernel before this one wrote them in ascending order, so the most
    // recently written ones, still in the last-level cache, are read first (4-5 % on this kernel in batched calls)
    const uint32_t zz = gridDim.z - 1 - blockIdx.z, comp = zz & 1u, item = zz >> 1, r = item / batch, b = item - r * batch;
    const uint64_t ct_limb = ((uint64_t)item * 2 + comp) * ell + i;
    const uint8_t *conv_limb = conv + ct_limb * LIMB, *acc_limb = acc + (((uint64_t)item * 2 + comp) * E + i) * LIMB;
    W* op = out + (uint64_t)b * out_bs + (uint64_t)r * out_rs + ((uint64_t)comp * out_limbs + i) * N;
    if constexpr (ADDEND == 2) {
        task_rows_finish<LOG_R, false, 2, W>(tw, mods[i], i, Pinv[i], addend_mul[i], conv_limb, acc_limb, op,
                                             static_cast<const uint8_t*>(addend) + ct_limb * LIMB, 1, rg, threadIdx.x, lds);
    } else if (ADDEND == 1 && comp == 0) {
        task_rows_finish<LOG_R, true, 1, W>(tw, mods[i], i, Pinv[i], 0.0, conv_limb, acc_limb, op,
                                            static_cast<const W*>(addend) + (uint64_t)b * addend_bs + (uint64_t)i * N, rot.galois[r], rg, threadIdx.x, lds);
    } else {
        task_rows_finish<LOG_R, false, 0, W>(tw, mods[i], i, Pinv[i], 0.0, conv_limb, acc_limb, op, nullptr, 1, rg, threadIdx.x, lds);
    }
}

void launch_rows_moddown_finish(const ks_ctx* c, const Level& lv, const uint8_t* acc, const uint8_t* conv, void* out_words, uint64_t out_bs,
                                const void* addend, uint64_t addend_bs, const MacRotations* rotations, uint64_t out_rs, uint32_t batch,
                                hipStream_t s, const FinishScale* fs, bool out_words32) {
    if (batch == 0) return;
    const double* mul = fs ? fs->mul : c->d_Pinv;
    const double* admul = fs ? fs->addend_mul : nullptr;
    const uint32_t out_limbs = fs ? fs->out_limbs : lv.ell, n_rot = rotations ? rotations->n : 1;
    if (out_limbs == 0) return;
    FinishRotations rot{};
    for (uint32_t r = 0; rotations && r < n_rot; ++r) rot.galois[r] = rotations->galois[r];
    const double wo = out_words32 ? 4.0 : 8.0;
    ProfScope ps("rows_moddown_finish", (double)batch * n_rot * out_limbs * (2 * 5 + 2 * 5 + 2 * wo + (!addend ? 0.0 : fs ? 10.0 : wo)) * c->N, s);
    const dim3 block(64), grid(c->N / 1024, out_limbs, batch * n_rot * 2);
#define KS_LAUNCH_FINISH(LOGR, MODE, WT)                                                                                        \
    hipLaunchKernelGGL((rows_moddown_finish<LOGR, MODE, WT>), grid, block, 0, s, c->tw_fwd, c->d_mod, mul, admul, lv.ell, lv.E, \
                       out_limbs, acc, conv, static_cast<WT*>(out_words), out_bs, out_rs, addend, addend_bs, batch, rot)
#define KS_LAUNCH_MODES(LOGR, WT)                       \
    if (fs) KS_LAUNCH_FINISH(LOGR, 2, WT);              \
    else if (addend) KS_LAUNCH_FINISH(LOGR, 1, WT);     \
    else KS_LAUNCH_FINISH(LOGR, 0, WT)
#define KS_LAUNCH(LOGR)                                   \
    if (out_words32) { KS_LAUNCH_MODES(LOGR, uint32_t); } \
    else { KS_LAUNCH_MODES(LOGR, uint64_t); }
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_MODES
#undef KS_LAUNCH_FINISH
}

// ------------------------------------------------------------------------------------------------
// Rescale.  The rescale's remainder r = (sum - conv)[ell-1] P^-1 (coefficient domain, centred) has to be subtracted from every
// other limb after the division by P: (acc_i - conv_i) P^-1 + d_i - r, times q_{ell-1}^-1.  As P r joins conv_i before the
// forward transform, it costs one more source of that conversion, and the rescale needs no transforms of its own (a
// forward transform and two more passes over every limb: 290 of 1310 us per 8 multiplications at L = 35).
// With y_k = [x_k (P / p_k)^-1]_{p_k} the converted special part of limb ell-1 times P^-1 is sum_k y_k p_k^-1.
// One thread per four coefficients, K + 1 sources read and one written.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rescale_remainder_kernel(Mod m, const double* __restrict__ pinv, uint32_t ell, uint32_t K,
                                                                uint32_t N, uint8_t* __restrict__ acc) {
    // quad t: rows 4 q .. 4 q + 3 of the 16 that the thread (r0, column) of the column kernels holds
    const uint32_t t = blockIdx.x * 256 + threadIdx.x, q = (t >> 8) & 3u;
    const uint64_t limb = packed_limb_bytes(N);
    const uint32_t bytes = 4 * N + source_bytes_offset(t >> 10, t & 255u) + 4 * q;
    uint8_t* last = acc + ((uint64_t)blockIdx.y * (ell + K) + ell - 1) * limb;
    const auto load = [&](const uint8_t* p, double (&v)[4]) {
        const Words4 lo = reinterpret_cast<const Words4*>(p)[t];
        const uint32_t top = *reinterpret_cast<const uint32_t*>(p + bytes);
#pragma unroll
        for (int x = 0; x < 4; ++x)   // canonical residues: the byte above is not negative
            v[x] = __builtin_bit_cast(double, (uint64_t)(0x43380000u | ((top >> (8 * x)) & 0xFFu)) << 32 | lo.w[x]) - kDigitBias;
    };
    static_assert(kMaxLimbsIn <= kMacTerms, "products per exact sum");
    double hi[4], lo[4], sum[4], r[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        hi[x] = kMacBias;
        lo[x] = 0.0;
    }
    load(last, sum);
#pragma unroll 4
    for (uint32_t k = 0; k < K; ++k) {
        double y[4];
        load(last + (uint64_t)(k + 1) * limb, y);
#pragma unroll
        for (int x = 0; x < 4; ++x) mac_exact(y[x], pinv[k], hi[x], lo[x]);
    }
    Words4 o;
    uint32_t h[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const double c = canon(reduce_lazy(sum[x] - mac_reduce(hi[x], lo[x], m), m), m);
        r[x] = c > (m.p - 1.0) * 0.5 ? c - m.p : c;
        const uint64_t bits = __builtin_bit_cast(uint64_t, r[x] + kDigitBias);
        o.w[x] = (uint32_t)bits;
        h[x] = (uint32_t)(bits >> 32);
    }
    reinterpret_cast<Words4*>(last)[t] = o;
    *reinterpret_cast<uint32_t*>(last + bytes) = low_bytes(h[0], h[1], h[2], h[3]);
}

void launch_rescale_remainder(const ks_ctx* c, const Level& lv, uint8_t* acc, uint32_t n_polys, hipStream_t s) {
    if (n_polys == 0) return;
    ProfScope ps("rescale_remainder", (double)n_polys * (c->K + 2) * packed_limb_bytes(c->N), s);
    const uint64_t q = c->mod[lv.ell - 1];
    hipLaunchKernelGGL(rescale_remainder_kernel, dim3(c->N / 1024, n_polys), dim3(256), 0, s, Mod{(double)q, 1.0 / (double)q}, lv.d_pinv_last,
                       lv.ell, c->K, c->N, acc);
}

}  // namespace ks
