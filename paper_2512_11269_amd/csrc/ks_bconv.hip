// Fast RNS base conversion with fp64 accumulation, for conversions of few sources to few targets (the others:
// ks_bconv_mfma.hip).
//
// A thread owns two adjacent coefficient positions, or one where the pieces of two would cost it occupancy.  It scales the residues to y_i = [x_i (D / s_i)^-1]_{s_i}, canonical, cuts
// them into the pieces of the fused conversion (split3, or split2 for moduli below 2^32) and then takes three (two) FMAs per
// source and target and one reduction per target.  Tables are uniform and come through scalar loads.  Bound by traffic.
#include "ks_internal.hpp"

namespace ks {

constexpr int positions(int n_src, int pieces) { return n_src * pieces <= 10 ? 2 : 1; }  // of a thread

// W: word type of in and out (strides in words)
template <int NSRC, int PIECES, typename W>
__global__ __launch_bounds__(256) void bconv_kernel(const BConvPlan* __restrict__ plans, const W* __restrict__ in, uint64_t in_ps,
                                                    W* __restrict__ out, uint64_t out_ps, uint32_t N) {
    constexpr int V = positions(NSRC, PIECES);
    struct alignas(V * sizeof(W)) Vec {
        W w[V];
    };
    const BConvPlan& P = plans[blockIdx.y];
    const uint32_t n = (blockIdx.x * 256 + threadIdx.x) * V;  // N is a multiple of 512
    const W* ip = in + (uint64_t)blockIdx.z * in_ps + n;
    W* op = out + (uint64_t)blockIdx.z * out_ps + n;
    const int n_src = (int)P.n_src, n_dst = (int)P.n_dst;
    Vec x[NSRC];
    // places past the last source repeat it against factors of zero: all tables and residues are requested at once
#pragma unroll
    for (int i = 0; i < NSRC; ++i) x[i] = *reinterpret_cast<const Vec*>(ip + (uint64_t)P.src_limb[min(i, n_src - 1)] * N);
    double y[NSRC][V][PIECES];
#pragma unroll
    for (int i = 0; i < NSRC; ++i)
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const Mod mi = P.src_mod[min(i, n_src - 1)];
            const double v = canon(mulmod_lazy(word_to_f64<W>(x[i].w[k]), P.src_inv[min(i, n_src - 1)], mi), mi);
            if constexpr (PIECES == 3) split3(v, y[i][k][2], y[i][k][1], y[i][k][0]);
            else split2(v, y[i][k][1], y[i][k][0]);
        }
#pragma unroll 1
    for (int t = 0; t < n_dst; ++t) {
        const Mod mt = P.dst_mod[t];
        double s[V] = {};
#pragma unroll
        for (int i = 0; i < NSRC; ++i)
#pragma unroll
            for (int p = PIECES - 1; p >= 0; --p)
#pragma unroll
                for (int k = 0; k < V; ++k) s[k] = __builtin_fma(y[i][k][p], P.hats[t][i][p], s[k]);
        Vec o;
#pragma unroll
        for (int k = 0; k < V; ++k) o.w[k] = f64_to_word<W>(canon(reduce_lazy(s[k], mt), mt));
        *reinterpret_cast<Vec*>(op + (uint64_t)P.dst_limb[t] * N) = o;
    }
}

void launch_bconv(const ks_ctx* c, const PlanSet& plans, uint32_t limbs_moved_per_poly, const void* in, uint64_t in_ps, void* out,
                  uint64_t out_ps, uint32_t n_polys, hipStream_t s, bool words32) {
    if (n_polys == 0 || plans.n_plans == 0) return;
    // Which kernel (KS_OPT_BCONV_KERNEL overrides).  The matrix cores take targets by six and cost little per source; this kernel
    // takes 9 instructions per target and one per source and piece, and few sources to scale.  Where the chip is full (before,
    // both are at the launch floor), 64 polynomials at N = 2^16, vector against matrix cores:
    //   28 bits: 1 -> 1 8.9 against 20.5 us, 1 -> 24 82 / 117, 3 -> 6 26 / 35, 5 -> 3 23 / 38, 5 -> 24 100 / 124, 8 -> 1 44 / 36; a
    // thread's walk over many targets shows where the chip is not full: 5 -> 24, one polynomial, 13.8 / 10.4 at best.
    //   36 bits, with the instructions per group of six: 1 -> 1 (12) 12.0 / 23.4, 1 -> 6 (72) 35.1 / 35.5, 1 -> 12 (72) 83 / 100,
    // 1 -> 24 160 / 147, 2 -> 4 (60) 30.9 / 32.4, 2 -> 6 (90) 40.2 / 40.5, 3 -> 4 (72) 36.0 / 39.0, 3 -> 5 (90) 41.2 / 40.5,
    // 4 -> 2 (42) 30.3 / 33.0, 5 -> 1 (24) 29.5 / 35.9, 5 -> 2 (48) 35.5 / 39.8, 8 -> 1 68 / 59.
    const uint32_t cost = plans.targets * (3 * plans.shape_src + 9);
    bool vector = plans.shape_src <= 5 && (plans.targets <= 12 || (uint64_t)n_polys * c->N >= 1u << 20);
    if (c->pieces == 3) vector &= cost <= (plans.shape_src <= 3 ? 72 : 50) * plans.sixes && plans.targets <= 12;
    const int kernel = c->opt[KS_OPT_BCONV_KERNEL] ? c->opt[KS_OPT_BCONV_KERNEL] : vector ? 1 : 2;
    if (kernel == 2) {
        launch_bconv_mfma(c, plans, limbs_moved_per_poly, in, in_ps, out, out_ps, n_polys, s, words32);
        return;
    }
    ProfScope ps("bconv", (double)limbs_moved_per_poly * n_polys * c->N * (words32 ? 4.0 : 8.0), s);
#define KS_LAUNCH_BCONV_W(NS, PC, WT)                                                                                             \
    hipLaunchKernelGGL((bconv_kernel<NS, PC, WT>), dim3(c->N / (256 * positions(NS, PC)), plans.n_plans, n_polys), dim3(256), 0, s,   \
                       plans.d_plans, static_cast<const WT*>(in), in_ps, static_cast<WT*>(out), out_ps, c->N)
#define KS_LAUNCH_BCONV(NS)                                      \
    if (words32) KS_LAUNCH_BCONV_W(NS, 2, uint32_t);             \
    else if (c->pieces == 2) KS_LAUNCH_BCONV_W(NS, 2, uint64_t); \
    else KS_LAUNCH_BCONV_W(NS, 3, uint64_t)
    if (plans.shape_src == 1) { KS_LAUNCH_BCONV(1); }
    else if (plans.shape_src == 2) { KS_LAUNCH_BCONV(2); }
    else if (plans.shape_src == 3) { KS_LAUNCH_BCONV(3); }
    else if (plans.shape_src == 4) { KS_LAUNCH_BCONV(4); }
    else if (plans.shape_src == 5) { KS_LAUNCH_BCONV(5); }
    else { KS_LAUNCH_BCONV(kMaxLimbsIn); }
#undef KS_LAUNCH_BCONV
#undef KS_LAUNCH_BCONV_W
}

}  // namespace ks
