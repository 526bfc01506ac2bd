// Gathers that hold the sums of several rows of diagonals, and gathers that meet the division (see ks_gather.hpp).
#include <algorithm>

#include "ks_gather.hpp"
#include "ks_tasks.hpp"

namespace ks {

// ------------------------------------------------------------------------------------------------
// Several rows of diagonals over the same rotations (the inner sums of a baby-step giant-step transform).  The rotated ciphertext of a
// baby step, sum_j sigma_b(digit_j) key_{b,j} (+ P sigma_b(c0)), is the same for every giant step: a thread forms it once for a slot, reduces
// it and multiplies it by the plaintext slots of `R` giant steps, whose sums it holds.  Keys and gathered slots, which are what
// rotate_mac_kernel reads, are then read once for R sums instead of for each.
//   Four rows of sixteen diagonals, eight ciphertexts, three digits, N = 2^16: 2280 us as four launches of rotate_mac_kernel, 1338; 28 bits
// 1668 -> 768.  What bounds it: traffic beyond the L2, 8.6 GB read and 0.7 written by the counters (6.9 TB/s), where keys (1.6 GB), plaintexts
// (1.1), slots (0.3) and sums once would be 3.7; the vector units are 62 % busy.
//   The sums of R = 4 rows take the registers that eight ciphertexts would: a wavefront takes up to four, and a bundle of more is two halves of its
// ciphertexts.  Of eight, 256 threads of a workgroup take either half, on the same slots and keys; of five to seven they are two launches.
// What a workgroup's rotations read again is the slots of one (position, part of the limb) for the ciphertexts of the launch: three digits of eight
// 3.5 MB for half of a limb of N = 2^16, 1.8 MB for a quarter (launch_rotate_mac_rows chooses).
//   Two wavefronts a SIMD do not hide a load of the next step (1684 us): with a set of operands for each digit, up to three, a load has the
// time of a whole rotation.
// ------------------------------------------------------------------------------------------------
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
    const GatherTile tile = gather_tile(E, logN, parts_log, threadIdx.x & 255u);
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
    // quarters of a limb where the slots of a half are more than an XCD's L2 of 4 MB keeps beside the streams, a crossover between measured sizes:
    // eight ciphertexts, N = 2^16, halves -> quarters, three digits (3.5 MB) 1472 -> 1393 us; 28 bits (3.1 MB) 768 -> 790, two digits (2.4 MB) 1350 -> 1336,
    // two ciphertexts 669 -> 677
    constexpr double kKeptSlots = 3.3 * (1 << 20);
    const bool large = lv.ndig * src.group * src_bytes(src) * (c->N / 2) > kKeptSlots;
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

// ------------------------------------------------------------------------------------------------
// The end of a group of hoisted rotations on the ciphertext limbs: out[r][b][c] = (sum_j sigma_r(src_j) key_r[j][c] - NTT_rows(conv[r][b][c]))
// P^-1 + [c = 0] sigma_r(c0[b]), canonical.  The sums meet the converted limbs in LDS and registers and never exist in memory, where they
// were 10 bytes a residue written and read again.
//   A workgroup owns four rows of one limb position for H ciphertexts (a half of a bundle of more than four, as above) and walks
// rotations of the group.  For each, a wavefront per ciphertext and component runs the row half of the converted limb's transform and
// leaves it in LDS; then every wavefront takes blocks of 64 slots, as the gathers do.  Two workgroups a compute unit (78 KB of LDS,
// 128 registers), so that one gathers while the other transforms.  Four rotations of eight ciphertexts, three digits, 24 limbs, N = 2^16: 494 us,
// where the two kernels took 243 + 418.  What bounds it: traffic, 2.0 GB read beyond the L2 and 0.8 written (5.6 TB/s), and the vector units, 55 % busy.
// ------------------------------------------------------------------------------------------------
// Wavefronts of a workgroup that holds H ciphertexts: eight for three as well, of which two only gather (sixteen blocks of 64 slots are three
// turns of six wavefronts but two of eight; 28 bits, five digits, 13 limbs, ten rotations of three 790 -> 581 us).
constexpr int finish_waves(int h) { return h == 3 ? 8 : 2 * h; }
struct RotateFinishArgs {
    TwTables tw;
    const Mod* mods;
    const double* Pinv;
    uint32_t ell, E, M, ndig;
    const uint8_t* conv;
    void* out;
    uint64_t out_bs;
    const void* c0;
    uint32_t per_group, half0;
};
template <int LOG_R, int H, int WAVES, typename W, bool PACKED, bool INT>
__device__ __forceinline__ void rotate_finish(const RotateFinishArgs& a, const GatherBundle& bundle, const MacRotations& rot, uint32_t pos, uint32_t rg,
                                              uint32_t half, double (*rows)[4 * kRowPitch], RowTwiddlesLds& tl) {
    using Sum = WideSum<INT>;
    using Factor = typename Sum::Factor;
    constexpr uint32_t N = 256u << LOG_R, R = 1u << LOG_R, LOGN = LOG_R + 8;
    constexpr uint64_t LIMB = packed_limb_bytes(N);
    // Blocks of 64 slots that a wavefront has in hand at once: one block of one ciphertext is too few loads in flight (28 bits, four digits,
    // 20 limbs, fourteen rotations, one block 572, four 465 us).
    constexpr int FEW = 16 / (H * WAVES), TILES = FEW > 4 ? 4 : FEW < 1 ? 1 : FEW;
    const uint32_t ell = a.ell, E = a.E, M = a.M, ndig = a.ndig;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u, j0 = lane & 15u, rr = lane >> 4;
    const bool transforms = 2 * H == WAVES || wave < 2 * H;   // uniform
    const Mod m = a.mods[pos];
    const double mul = a.Pinv[pos];
    const uint64_t slots = (uint64_t)ndig * E * N;
    const uint32_t hi_bytes = gather_hi_bytes(bundle.group);
    const HalfSource src{uniform_rsrc(bundle.lo, slots * 4 * bundle.group), uniform_rsrc(bundle.hi, PACKED ? slots * hi_bytes : 0), bundle.group, half, hi_bytes};
    // the converted limb of this wavefront: ciphertext wave / 2 of the half, component wave % 2
    const uint8_t* cv = a.conv + ((uint64_t)(half * 8 + (transforms ? wave : 0)) * ell + pos) * LIMB;
    const uint64_t cv_rs = (uint64_t)bundle.group * 2 * ell * LIMB;
    const uint32_t r_first = blockIdx.y * a.per_group, r_last = min(r_first + a.per_group, rot.n) - 1;
    PackedRaw raw = packed_load<64>(cv + r_first * cv_rs, N, rg * 256 + lane);
    if (wave == 0) store_row_twiddles(tl.ta, tl.tb, a.tw, pos, N, R + rg * 4 + rr, lane, m);
    __syncthreads();
#pragma unroll 1
    for (uint32_t r = r_first; r <= r_last; ++r) {
        if (transforms) {
            double* lrow = rows[wave] + rr * kRowPitch;
            double w[16];
            unpack_rows(raw, w);
            uint32_t from = lane;
            asm volatile("" : "+v"(from));   // the offset is formed anew: kept across the loop it spills
            raw = packed_load<64>(cv + min(r + 1, r_last) * cv_rs, N, rg * 256 + from);
            uint32_t ta_at = rr * 16, tb_at = lane;
            asm volatile("" : "+v"(ta_at), "+v"(tb_at));   // the twiddles stay in LDS: hoisted out of the loop they take sixty registers
            radix16_fwd_lds(w, tl.ta + ta_at, 1, m);
#pragma unroll
            for (int k = 0; k < 16; ++k) lrow[j0 + 17 * k] = w[k];
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < 16; ++k) w[k] = lrow[17 * j0 + k];
            radix16_fwd_lds(w, tl.tb + tb_at - 64, 64, m);
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < 16; ++k) lrow[17 * j0 + k] = w[k];
        }
        __syncthreads();
        // a key is below 4 GB: [8][2][255][2^16] words of at most 8 bytes
        const BufferRsrc key = uniform_rsrc(rot.key[r], (uint64_t)ndig * 2 * M * N * sizeof(W));
        const uint32_t g = rot.galois[r];
#pragma unroll 1
        for (uint32_t tile = wave; tile < 16; tile += TILES * WAVES) {
            struct Raw {
                HalfRaw<H> x[TILES];
                W k0[TILES], k1[TILES];
            };
            uint32_t n[TILES], sn[TILES];
#pragma unroll
            for (int i = 0; i < TILES; ++i) {
                n[i] = rg * 1024 + (tile + i * WAVES) * 64 + lane;
                sn[i] = galois_source_slot(n[i], g, LOGN);
            }
            const auto fetch = [&](uint32_t j) {
                Raw q;
                const uint32_t limb = (j * 2 * M + pos) * N * (uint32_t)sizeof(W);
#pragma unroll
                for (int i = 0; i < TILES; ++i) {
                    q.x[i] = half_load<H, PACKED>(src, j * E + pos, N, sn[i]);
                    q.k0[i] = buffer_load<W>(key, n[i] * (uint32_t)sizeof(W), limb);
                    q.k1[i] = buffer_load<W>(key, n[i] * (uint32_t)sizeof(W), limb + M * N * (uint32_t)sizeof(W));
                }
                return q;
            };
            Raw cur = fetch(0);
            W add[TILES][H];
            Sum t[TILES][2 * H];
#pragma unroll
            for (int i = 0; i < TILES; ++i) {
#pragma unroll
                for (int b = 0; b < H; ++b)
                    add[i][b] = static_cast<const W*>(a.c0)[(uint64_t)(half * 4 + b) * (2ull * ell * N) + (uint64_t)pos * N + sn[i]];
#pragma unroll
                for (int b = 0; b < 2 * H; ++b) t[i][b].start(0.0);
            }
#pragma unroll 1
            for (uint32_t j = 0; j < ndig; ++j) {
                const Raw next = fetch(min(j + 1, ndig - 1));
#pragma unroll
                for (int i = 0; i < TILES; ++i) {
                    const Factor k0 = Sum::word(cur.k0[i]), k1 = Sum::word(cur.k1[i]);
                    Factor x[H];
                    half_take<H, PACKED, INT>(src, cur.x[i], x);
#pragma unroll
                    for (int b = 0; b < H; ++b) {
                        t[i][2 * b].add(x[b], k0);
                        t[i][2 * b + 1].add(x[b], k1);
                    }
                }
                cur = next;
            }
#pragma unroll
            for (int i = 0; i < TILES; ++i) {
                const uint32_t at = n[i] & 1023u, p = at & 255u, in_row = (at >> 8) * kRowPitch + p + (p >> 4);
                W* op = static_cast<W*>(a.out) + (uint64_t)(half * 4) * a.out_bs + (uint64_t)r * (2ull * ell * N) + (uint64_t)pos * N + n[i];
#pragma unroll
                for (int b = 0; b < 2 * H; ++b) {
                    double v = mulmod_lazy(t[i][b].result(m) - rows[b][in_row], mul, m);
                    if (b % 2 == 0) v = reduce_lazy(v + word_to_f64<W>(add[i][b / 2]), m);
                    op[(uint64_t)(b / 2) * a.out_bs + (b & 1) * ((uint64_t)ell * N)] = f64_to_word<W>(canon(v, m));
                }
            }
        }
        __syncthreads();   // the converted limbs have been read
    }
}
// H: ciphertexts of the first half, HB: of the second (0: this launch has the half half0 alone).  Both halves in one launch, next to each other:
// the second finds the keys in cache (six ciphertexts, two digits, four limbs, eight rotations 356 us in two launches, 320 in one).
template <int LOG_R, int H, int HB, typename W, bool PACKED, bool INT>
__global__ __launch_bounds__(64 * finish_waves(H), H >= 3 ? 4 : 3) void rotate_finish_kernel(RotateFinishArgs a, uint32_t parts_log, GatherBundle bundle,
                                                                                              MacRotations rot) {
    constexpr uint32_t LOGN = LOG_R + 8, HALVES = HB ? 2 : 1;
    __shared__ double rows[2 * H][4 * kRowPitch];
    __shared__ RowTwiddlesLds tl;
    // gather_tile with 1024 slots, the halves of a tile next to each other
    const uint32_t per_unit = 1u << (LOGN - 10 - parts_log), turn = blockIdx.x >> 3, local = turn / HALVES, half = turn % HALVES;
    const uint32_t unit = (local / per_unit) * 8 + (blockIdx.x & 7);
    if (unit >= (a.ell << parts_log)) return;  // uniform
    uint32_t pos = unit >> parts_log, rg = (unit & ((1u << parts_log) - 1)) * per_unit + local % per_unit;
    if (HB == 0 || HB == H || half == 0) {  // uniform
        rotate_finish<LOG_R, H, finish_waves(H), W, PACKED, INT>(a, bundle, rot, pos, rg, HB == 0 ? a.half0 : HB == H ? half : 0, rows, tl);
    } else if constexpr (HB != 0) {
        asm volatile("" : "+s"(pos), "+s"(rg));   // nothing of this half is computed ahead of the branch
        rotate_finish<LOG_R, HB, finish_waves(H), W, PACKED, INT>(a, bundle, rot, pos, rg, 1, rows, tl);
    }
}

// Wavefronts with work decide, one per rotation, ciphertext, component and four rows; many digits and few ciphertexts make a rotation's
// gathers, which the sums in memory run at more wavefronts a SIMD, the longer part.  Calls with the sums in memory -> meeting the division, us,
// N = 2^16, 24 limbs, three digits, sixteen rotations: one ciphertext 863 -> 805 (24576 wavefronts), two 1330 -> 1187, three 1858 -> 1678,
// four 2480 -> 2153, six 3688 -> 3289, seven 4264 -> 3686, eight 4818 -> 4159 (98304); 28 bits, one 644 -> 560, five 2625 -> 2326, eight 4143 -> 3459.
//   Line: one ciphertext, N = 2^16, 12 limbs (9216) 342 -> 310, but six, N = 2^15, 7 limbs, four digits (16128) 245 -> 254.  Below N = 2^15, where
// keys and slots stay in cache: two digits, 9 limbs, seven ciphertexts (18144) 928 -> 925, three, 9 limbs, eight (18432) 250 -> 261, four, 14 limbs,
// seven (25088) 1218 -> 1123, five, 13 limbs, eight (29952) 743 -> 782.  Five ciphertexts are two launches, the second for one: two digits, 7 limbs
// (17920) 653 -> 668, 8 limbs (20480) 816 -> 804, 17 limbs (43520) 1354 -> 1312; three, 21 limbs (53760) 880 -> 865; five, 13 limbs (33280)
// 877 -> 976.  Six, six digits, 17 limbs (52224) 1495 -> 1549.
bool rotations_meet_division(const ks_ctx* c, const Level& lv, uint32_t group, uint32_t n_rot) {
    const uint32_t wavefronts = lv.ell * (c->N / 1024) * 2 * group * n_rot;
    const uint32_t most = group == 5 ? 3 : group == 6 ? 5 : kMaxDigits;
    if (c->logN < 15) return wavefronts > (lv.ndig <= 2 ? 16384 : 22000) && lv.ndig <= std::min(most, 4u);
    return wavefronts > (group == 5 ? 20000 : 16384) && lv.ndig <= most;
}

void launch_rotate_finish(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, const uint8_t* conv, void* out,
                          uint64_t out_bs, const void* c0, hipStream_t s, bool words32) {
    if (rot.n == 0) return;
    const uint32_t pl = std::min(lv.ell % 4 == 1 || lv.ell % 4 == 2 ? 2u : 1u, c->logN - 10);
    const double wk = words32 ? 4.0 : 8.0;
    ProfScope ps("rotate_finish", (src_bytes(src) * src.group * lv.ndig + (double)rot.n * (wk * 2.0 * lv.ndig + (10.0 + 3.0 * wk) * src.group)) * lv.ell * c->N, s);
    const uint32_t grid = ((lv.ell << pl) + 7) / 8 * 8 * ((c->N / 1024) >> pl);
    const bool ints = !src.hi && integer_sums(c);
    // Rotations that a workgroup walks: the next one's converted limb is requested early and the twiddles stay, which saves about a quarter of
    // a rotation each time (eight ciphertexts, N = 2^16, 24 limbs, 3072 workgroups, all of four 4181 us, two 4240, one 4409), but a launch of
    // few rounds of workgroups (up to six, three or two a compute unit by their LDS) ends in half a round on average.  All of them unless
    // fewer are clearly ahead (one ciphertext, 27 limbs, 1728, all of five rotations 424 us, one 368; four, N = 2^15, 20 limbs, 640, all of
    // eight 512, two 491; eight, N = 2^15, 26 limbs, 1664, all of five 885, one 919).
    const auto rotations = [&](int h, uint32_t halves) {
        const uint32_t workgroups = grid * halves, resident = 256 * (h == 1 ? 6 : h == 2 ? 3 : 2);
        const auto cost = [&](uint32_t per) { return (2 * workgroups * ((rot.n + per - 1) / per) + resident) * (4 * per + 1); };
        uint32_t best = rot.n;
        for (uint32_t per = rot.n; per > 0; --per)
            if (cost(per) < cost(best)) best = per;
        return 40 * cost(best) < 39 * cost(rot.n) ? best : rot.n;
    };
    RotateFinishArgs a{c->tw_fwd, c->d_mod, c->d_Pinv, lv.ell, lv.E, c->M, lv.ndig, conv, out, out_bs, c0, 0, 0};
#define KS_LAUNCH_RF(LOGR, HV, HBV, WT, PK, IS)                                                                                               \
    a.per_group = rotations(HV, (HBV) ? 2 : 1);                                                                                               \
    hipLaunchKernelGGL((rotate_finish_kernel<LOGR, HV, HBV, WT, PK, IS>),                                                                     \
                       dim3(grid * ((HBV) ? 2 : 1), (rot.n + a.per_group - 1) / a.per_group), dim3(64 * finish_waves(HV)), 0, s, a, pl, src, rot)
#define KS_LAUNCH_H(LOGR, HV, HBV)                                               \
    {                                                                            \
        if (ints) { KS_LAUNCH_RF(LOGR, HV, HBV, uint32_t, false, true); }        \
        else if (words32) { KS_LAUNCH_RF(LOGR, HV, HBV, uint32_t, false, false); } \
        else { KS_LAUNCH_RF(LOGR, HV, HBV, uint64_t, true, false); }             \
    }
#define KS_LAUNCH(LOGR)                           \
    switch (src.group) {                          \
        case 1: KS_LAUNCH_H(LOGR, 1, 0) break;    \
        case 2: KS_LAUNCH_H(LOGR, 2, 0) break;    \
        case 3: KS_LAUNCH_H(LOGR, 3, 0) break;    \
        case 4: KS_LAUNCH_H(LOGR, 4, 0) break;    \
        case 5: KS_LAUNCH_H(LOGR, 4, 0)           \
            a.half0 = 1;                          \
            KS_LAUNCH_H(LOGR, 1, 0) break;        \
        case 6: KS_LAUNCH_H(LOGR, 4, 2) break;    \
        case 7: KS_LAUNCH_H(LOGR, 4, 3) break;    \
        default: KS_LAUNCH_H(LOGR, 4, 4) break;   \
    }
    KS_FOR_LOG_R(c->logN, KS_LAUNCH)
#undef KS_LAUNCH
#undef KS_LAUNCH_H
#undef KS_LAUNCH_RF
}

}  // namespace ks
