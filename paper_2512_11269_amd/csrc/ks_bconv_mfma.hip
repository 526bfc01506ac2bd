// Base conversion on the matrix cores (int8 MFMA), fused with the column half of the forward transform of every target
// limb (Kernel Code Generation: "Base Conversion" kernel class; the tensor-core formulations in the paper's Related Work).
//
// The conversion sum  out_t = sum_i y_i (D / s_i)  (mod t)  is a contraction over the sources i with one modulus per
// output column, so it cannot run on the matrix cores as it stands.  Cut into bytes it can: y_i = sum_a d_{i,a} 256^a
// with five signed digits d (|d| <= 128), and for every digit position the factor [(D / s_i) 256^a]_t, centred, is cut
// the same way into digits e_{t,i,a,b}.  Then
//     y_i (D / s_i) = sum_b 256^b  S_b   (mod t),     S_b = sum_{i,a} d_{i,a} e_{t,i,a,b},
// and the five S_b of a target are dot products of length 5 n_src over small integers: one row of an int8 matrix
// product with exact 32-bit accumulation (|S_b| <= 17 * 5 * 2^14).  The recombined value is below 2^49 in magnitude,
// exact in a double, and one Barrett step makes it a lazy residue modulo t.
//
// v_mfma_i32_32x32x32_i8: every lane supplies 16 bytes of A (row = lane % 32) and 16 bytes of B (column = lane % 32) for
// the 16 contraction indices of its half (lane / 32); result register j of a lane holds row 8 (j / 4) + 4 (lane / 32) + j % 4
// of its column.  Here a COLUMN IS A COEFFICIENT POSITION, so the B operand of a lane is made of the bytes of that lane's
// own source residues: no data crosses lanes on the way in.  The two lanes that share a column (l and l + 32) read
// different sources and receive different targets: rows are ordered so that result registers 5 u + b of a lane are the
// five digit planes b of its u-th target.  A workgroup owns a tile of 2048 positions (4096 with eight wavefronts) and 2 TL targets (TL per lane half):
// thread (pair p = 32 wave + lane % 32, half h) walks the 16 positions (row r0 + 16 k, column c) of pair p, exactly the
// points the column butterflies need in its registers afterwards.
#include "ks_internal.hpp"
#include "ks_tasks.hpp"

namespace ks {

// Workgroups per compute unit the register allocation must leave room for: without a bound the scheduler hoists the
// matrix instructions of all 16 positions (256 result registers) and the kernel drops to one wavefront per SIMD.
// Four where the registers of one target fit into 128: nine sources a half need more and, as four workgroups, spilled 22
// (key-switch 15 -> 30 moduli, N = 2^16: 116.0 us, three 108.2; 15 -> 15 at N = 2^15 53.8 and 50.3; seven sources a half are
// 1 % ahead with four).
constexpr int mfma_min_blocks(int tl, int t) { return tl == 1 ? (t <= 7 ? 4 : 3) : 2; }

template <int LOG_R, int TL, int T, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 4 ? mfma_min_blocks(TL, T) : 1) void bconv_mfma_ntt_cols(const double* __restrict__ tw, const BConvPlan* __restrict__ plans,
                                                           LaunchMeta meta, const uint8_t* __restrict__ y, uint64_t y_ps,
                                                           uint8_t* __restrict__ out, uint64_t out_ps, uint32_t n_polys, uint32_t n_subsets, uint32_t pair) {
    using Shape = MfmaConvShape<LOG_R, TL, WAVES>;
    __shared__ double lds[Shape::LDS_WORDS];
    __shared__ double lds_tw[Shape::LDS_TW_WORDS];
    const uint32_t plan_id = blockIdx.y / n_subsets, subset = blockIdx.y - plan_id * n_subsets;
    const PlanMeta& PM = meta.plan[plan_id];  // kernel arguments: scalar loads, nothing else to wait for
    const int t0 = (int)subset * 2 * TL;
    if (t0 >= (int)PM.n_dst) return;  // uniform for the whole workgroup
    uint32_t tile = blockIdx.x;
    // Tiles of 8 columns are half a 128-byte line wide.  Workgroup ids x and x + 8 run on the same XCD at about the same time:
    // they take the two halves of a line, so that its second half is read from, and its stores meet in, that XCD's L2 (eight
    // ciphertexts, L = 35: 438 -> 386 us of conversions).  Not where one round holds the whole launch: there the second fetch is
    // served by the memory-side cache and pairing cost the single-ciphertext key-switch 1.3 % (106.2 -> 107.6 us).
    if (Shape::TC == 8 && pair) tile = (tile & ~15u) | ((tile & 7u) << 1) | ((tile >> 3) & 1u);
    task_bconv_mfma_cols<LOG_R, TL, T, WAVES>(tw, plans[plan_id], PM, y, y_ps, out, out_ps, blockIdx.z, gridDim.z, n_polys, tile, t0,
                                                    threadIdx.x, lds, lds_tw);
}

// Targets per lane half: one gives the most workgroups, three shares the byte-cutting of the sources among the most
// targets (and keeps the stores of one target under the butterflies of the next).  wide: tiles of 16 columns and 512 threads
// instead of 8 and 256 at N = 2^16, whole 128-byte lines, for launches of many rounds and many sources (conversion_tile).
void launch_bconv_mfma_ntt_cols(const ks_ctx* c, const PlanSet& plans, const uint8_t* y, uint64_t y_ps, uint8_t* out,
                                uint64_t out_ps, uint32_t n_polys, int tl, bool wide, hipStream_t s) {
    const uint32_t n_src = plans.shape_src, n_plans = plans.n_plans, max_targets = plans.max_targets;
    const BConvPlan* d_plans = plans.d_plans;
    const uint32_t t = mfma_sources(n_src);
    tl = (c->logN == 13 || c->logN == 14) || tl < 2 ? 1 : 3;  // built shapes: one or three targets per lane half
    const int waves = wide && c->logN == 16 && tl == 3 && n_src > 4 ? 8 : 4;
    const uint32_t tiles = c->N / (512 * waves);
    const uint32_t n_subsets = (max_targets + 2 * tl - 1) / (2 * tl);
    // Polynomials that a workgroup takes in turn, up to eight: each round of workgroups (one to four per compute unit) takes about as
    // long as another, and a polynomial after
    // the first an eighth less (its sources arrive under the butterflies of the one before; factors and twiddles are there): four hoisted
    // rotations of eight ciphertexts, 64 polynomials 8 -> 24, 269 -> 241 us; 16 polynomials 90 -> 84; 13 -> 34 136 -> 133.
    // Three targets a half pay for the loop with spilled registers: 2 to 4 with four sources a half, 4 to 6 with seven, 17 or 18 with nine.
    // Forming the lanes' places anew for every polynomial takes those of four away and most of the others', but is slower: sixteen
    // rotations -0.7 %, key-switches 12 -> 36 x 8 717 -> 728 us, 13 -> 39 x 4 438 -> 450, 14 -> 28 x 8 538 -> 553, 15 -> 30 x 8 569 -> 596.
    const uint32_t slots = waves == 8 ? 256 : 256 * mfma_min_blocks(tl, (int)t), per_poly = tiles * n_plans * n_subsets;
    uint32_t groups = n_polys;
    double least = 1e30;
    for (uint32_t z = (n_polys + 7) / 8; z <= n_polys; ++z) {
        const uint32_t items = (n_polys + z - 1) / z;
        const double rounds = (double)(((uint64_t)per_poly * z + slots - 1) / slots), cost = rounds * (1.0 + 0.88 * (items - 1));
        if (cost < least) {
            least = cost;
            groups = z;
        }
    }
    const dim3 grid(tiles, n_plans * n_subsets, groups), block(64 * waves);
#define KS_LAUNCH_MFMA(LOGR, TLV, TV, WV)                                                                                            \
    hipLaunchKernelGGL((bconv_mfma_ntt_cols<LOGR, TLV, TV, WV>), grid, block, 0, s, c->d_tw_fwd, d_plans, plans.meta, y, y_ps, \
                       out, out_ps, n_polys, n_subsets, tiles * n_plans * n_subsets * n_polys > 512)
#define KS_MFMA_SHAPE(LOGR, TLV)                           \
    switch (t) {                                           \
        case 1: KS_LAUNCH_MFMA(LOGR, TLV, 1, 4); break;    \
        case 2: KS_LAUNCH_MFMA(LOGR, TLV, 2, 4); break;    \
        case 3: KS_LAUNCH_MFMA(LOGR, TLV, 3, 4); break;    \
        case 4: KS_LAUNCH_MFMA(LOGR, TLV, 4, 4); break;    \
        case 6: KS_LAUNCH_MFMA(LOGR, TLV, 6, 4); break;    \
        case 7: KS_LAUNCH_MFMA(LOGR, TLV, 7, 4); break;    \
        default: KS_LAUNCH_MFMA(LOGR, TLV, 9, 4); break;   \
    }
#define KS_LAUNCH_TL(LOGR)                       \
    {                                            \
        if (tl == 1) { KS_MFMA_SHAPE(LOGR, 1); } \
        else { KS_MFMA_SHAPE(LOGR, 3); }         \
    }
    // every shape for the degrees that conversion_tile takes here and for the smallest one (which the parity
    // sweeps run on); the degrees in between take one target per lane half
    switch (c->logN) {
        case 12: KS_LAUNCH_TL(4) break;
        case 13: KS_MFMA_SHAPE(5, 1); break;
        case 14: KS_MFMA_SHAPE(6, 1); break;
        case 15: KS_LAUNCH_TL(7) break;
        default:
            if (waves == 4) KS_LAUNCH_TL(8)
            else if (t == 3) KS_LAUNCH_MFMA(8, 3, 3, 8);
            else if (t == 4) KS_LAUNCH_MFMA(8, 3, 4, 8);
            else if (t == 6) KS_LAUNCH_MFMA(8, 3, 6, 8);
            else if (t == 7) KS_LAUNCH_MFMA(8, 3, 7, 8);
            else KS_LAUNCH_MFMA(8, 3, 9, 8);
            break;
    }
#undef KS_LAUNCH_TL
#undef KS_MFMA_SHAPE
#undef KS_LAUNCH_MFMA
}

// ------------------------------------------------------------------------------------------------
// Standalone conversion on the matrix cores (the `bconv` entry point but for few sources): canonical residues in, canonical residues out, no
// transform.  A wavefront owns PG groups of 32 positions, V of them interleaved so that a lane's V positions are one 16-byte
// access: lane (position l % 32, half l / 32) scales its slots' source residues to y_i = [x_i (D / s_i)^-1]_{s_i}, cuts them
// into bytes once, and then walks the targets six at a time (three per lane half), writing 512-byte segments per target.  The factors and
// constants of the next six targets are requested before the current ones' stores: loads and stores share one in-order counter, so a load behind the
// stores would wait for memory to acknowledge them.  About 16 vector instructions per position and target remain, where
// fp64 accumulation takes three per source more; what bounds a full launch is the traffic itself:
// 24 polynomials, 12 -> 35 moduli, N = 2^16: 118 us = 5.0 TB/s (64: 5.4), where fp64 accumulation of 12-bit pieces took
// 187; in 32-bit words 76 against 162; calls of one polynomial, 8 -> 24: 11.9 against 18.6.  Few sources: ks_bconv.hip.
// ------------------------------------------------------------------------------------------------
template <int T, int PG, typename W>
__global__ __launch_bounds__(256) void bconv_mfma_kernel(const BConvPlan* __restrict__ plans, LaunchMeta meta,
                                                         const W* __restrict__ in, uint64_t in_ps,
                                                         W* __restrict__ out, uint64_t out_ps, uint32_t N) {
    constexpr int NM = mfma_instructions(T);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, h = lane >> 5;
    constexpr int V = PG * (int)sizeof(W) <= 16 ? PG : 16 / (int)sizeof(W);
    struct alignas(V * sizeof(W)) Vec {
        W w[V];
    };
    const uint32_t n = (blockIdx.x * 4 + (tid >> 6)) * (32 * PG) + (lane & 31u) * V;  // N is a multiple of 128 PG
    const BConvPlan& P = plans[blockIdx.y];
    const int n_dst = (int)meta.plan[blockIdx.y].n_dst, n_src = (int)P.n_src;
    const W* ip = in + (uint64_t)blockIdx.z * in_ps + n;
    W* op = out + (uint64_t)blockIdx.z * out_ps + n;
    W xraw[PG][T];
    Mod mi[T];
    double inv[T];
#pragma unroll
    for (int e = 0; e < T; ++e) {
        const int i = min(2 * e + (int)h, n_src - 1);  // places past the last source repeat it against zero factors
        const W* src = ip + (uint64_t)P.src_limb[i] * N;
#pragma unroll
        for (int g = 0; g < PG; g += V) {
            const Vec v = *reinterpret_cast<const Vec*>(src + 32 * g);
#pragma unroll
            for (int k = 0; k < V; ++k) xraw[g + k][e] = v.w[k];
        }
        mi[e] = P.src_mod[i];
        inv[e] = P.src_inv[i];
    }
    // row r of the factor matrix: result register 4 (r / 8) + r % 4 of lane half (r / 4) % 2, i.e. digit plane b of that
    // half's target ua
    const uint32_t r = lane & 31u, hp = (r >> 2) & 1u, j = 4 * (r >> 3) + (r & 3u), ua = min(j / 5, 2u), b = min(j - 5 * ua, 4u);
    v4i afac[NM];
    BConvPlan::TargetRec rec[3];
    auto request = [&](int t0) {
        const int ta = min(t0 + (int)(hp * 3 + ua), n_dst - 1);  // (register 15 is unused: it repeats a valid row)
#pragma unroll
        for (int m = 0; m < NM; ++m) afac[m] = *reinterpret_cast<const v4i*>(&P.afac[ta][b][2 * m + h][0]);
#pragma unroll
        for (int u = 0; u < 3; ++u) rec[u] = P.trec[min(t0 + (int)h * 3 + u, n_dst - 1)];
    };
    request(0);
    v4i bq[PG][NM];
#pragma unroll
    for (int g = 0; g < PG; ++g)
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            bq[g][m] = v4i{0, 0, 0, 0};
            uint32_t top = 0;
#pragma unroll
            for (int e = 0; e < mfma_slot_sources(T, m); ++e) {
                const int i = mfma_slot_start(T, m) + e;
                const double yi = canon(mulmod_lazy(word_to_f64<W>(xraw[g][i]), inv[i], mi[i]), mi[i]);
                const uint64_t bits = __builtin_bit_cast(uint64_t, yi + kDigitBias);
                bq[g][m][e] = (int)((uint32_t)bits ^ 0x80808080u);
                top |= ((uint32_t)(bits >> 32) & 0xFFu) << (8 * e);
            }
            bq[g][m][3] = (int)top;
        }
#pragma unroll 1
    for (int t0 = 0; t0 < n_dst; t0 += 6) {
        v16i s[PG];
#pragma unroll
        for (int g = 0; g < PG; ++g) {
            s[g] = v16i{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int m = 0; m < NM; ++m) s[g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(afac[m], bq[g][m], s[g], 0, 0, 0);
        }
        Mod mt[3];
        uint32_t limb[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            mt[u] = rec[u].m;
            limb[u] = rec[u].limb;
        }
        request(t0 + 6);  // past the end: the last target again
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (t0 + (int)h * 3 + u < n_dst) {
                W* dst = op + (uint64_t)limb[u] * N;
#pragma unroll
                for (int g = 0; g < PG; g += V) {
                    Vec o;
#pragma unroll
                    for (int k = 0; k < V; ++k) {
                        const v16i& q = s[g + k];
                        const int lo = q[5 * u] + (q[5 * u + 1] << 8), mid = q[5 * u + 2] + (q[5 * u + 3] << 8);
                        const double v = __builtin_fma((double)q[5 * u + 4], 4294967296.0, __builtin_fma((double)mid, 65536.0, (double)lo));
                        o.w[k] = f64_to_word<W>(canon(reduce_lazy(v, mt[u]), mt[u]));
                    }
                    *reinterpret_cast<Vec*>(dst + 32 * g) = o;
                }
            }
        }
    }
}

void launch_bconv_mfma(const ks_ctx* c, const PlanSet& plans, uint32_t limbs_moved_per_poly, const void* in, uint64_t in_ps,
                       void* out, uint64_t out_ps, uint32_t n_polys, hipStream_t s, bool words32) {
    if (n_polys == 0 || plans.n_plans == 0) return;
    const uint32_t t = mfma_sources(plans.shape_src);
    // position groups per wavefront: more of them share the factor loads of a step and widen the accesses, as long as the
    // launch still fills the chip (256 compute units) a few times over
    const uint64_t tiles = (uint64_t)n_polys * plans.n_plans * (c->N / 128);
    const int pg = tiles / 4 >= 1024 ? 4 : tiles / 2 >= 512 ? 2 : 1;
    const dim3 grid(c->N / (128 * pg), plans.n_plans, n_polys), block(256);
    ProfScope ps("bconv_mfma", (double)limbs_moved_per_poly * n_polys * c->N * (words32 ? 4.0 : 8.0), s);
#define KS_LAUNCH_BM_W(TV, PGV, WT)                                                                                                  \
    hipLaunchKernelGGL((bconv_mfma_kernel<TV, PGV, WT>), grid, block, 0, s, plans.d_plans, plans.meta, static_cast<const WT*>(in), in_ps, \
                       static_cast<WT*>(out), out_ps, c->N)
#define KS_LAUNCH_BM_PG(TV, WT)                        \
    if (pg == 4) KS_LAUNCH_BM_W(TV, 4, WT);            \
    else if (pg == 2) KS_LAUNCH_BM_W(TV, 2, WT);       \
    else KS_LAUNCH_BM_W(TV, 1, WT)
#define KS_LAUNCH_BM(TV)                                       \
    {                                                                 \
        if (words32) { KS_LAUNCH_BM_PG(TV, uint32_t); }        \
        else { KS_LAUNCH_BM_PG(TV, uint64_t); }                \
    }
    if (t == 1) KS_LAUNCH_BM(1)
    else if (t == 2) KS_LAUNCH_BM(2)
    else if (t == 3) KS_LAUNCH_BM(3)
    else if (t == 4) KS_LAUNCH_BM(4)
    else if (t == 6) KS_LAUNCH_BM(6)
    else if (t == 7) KS_LAUNCH_BM(7)
    else KS_LAUNCH_BM(9)
#undef KS_LAUNCH_BM
#undef KS_LAUNCH_BM_PG
#undef KS_LAUNCH_BM_W
}

}  // namespace ks
