// Internal declarations shared by the translation units of the library (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <mutex>
#include <type_traits>
#include <vector>

#include "../../include/ks.h"
#include "ks_device.hpp"
#include "ks_tiles.hpp"

namespace ks {

constexpr int kMaxLimbsIn = 16; // source limbs a caller may ask for (alpha, K, bconv)
constexpr int kMaxSrc = 18;     // source slots of a conversion plan: kMaxLimbsIn, the dropped limb of a rescale, one of padding
constexpr int kMfmaSlots = 6;   // 16-byte operand slots of the matrix-core conversion: 3 instructions x 2 lane halves, 3 sources each
// Sources per lane half of the matrix-core conversion, of those it is built for; instructions per position; sources of instruction m and
// the first of them (dealt evenly).
constexpr uint32_t mfma_sources(uint32_t n_src) { return n_src <= 8 ? (n_src + 1) / 2 : n_src <= 12 ? 6 : n_src <= 14 ? 7 : 9; }
constexpr int mfma_instructions(int t) { return (t + 2) / 3; }
constexpr int mfma_slot_sources(int t, int m) { return (t + mfma_instructions(t) - 1 - m) / mfma_instructions(t); }
constexpr int mfma_slot_start(int t, int m) { return m == 0 ? 0 : mfma_slot_start(t, m - 1) + mfma_slot_sources(t, m - 1); }
constexpr int mfma_slot_of(int t, int e) { return e < mfma_slot_sources(t, 0) ? 0 : e < mfma_slot_start(t, 2) ? 1 : 2; }
constexpr int kMfmaPlanes = 5;  // signed base-256 digits of a 36-bit residue or factor
constexpr int kMaxDst = 256;    // target limbs of one base conversion
constexpr int kMaxLimbs = 192;  // limbs of one polynomial bundle addressed by a LimbMap
constexpr int kMaxDigits = 8;

// Which limbs of a polynomial bundle a transform launch touches: limb `idx` lives at element offset
// off[idx] * N from the bundle's base and is taken modulo moduli[mod[idx]].  Passed by value.
struct LimbMap {
    uint16_t off[kMaxLimbs];
    uint8_t mod[kMaxLimbs];
    uint32_t n;
};

// Constants of one fast base conversion, read by the kernel through uniform (scalar) loads.
struct BConvPlan {
    uint32_t n_src, n_dst;
    uint32_t src_limb[kMaxSrc];  // limb index inside the input bundle (32-bit fields: scalar loads)
    uint32_t dst_limb[kMaxDst];  // limb index inside the output bundle
    Mod src_mod[kMaxSrc];
    double src_inv[kMaxSrc];     // (D / s_i)^-1 mod s_i
    Mod dst_mod[kMaxDst];
    uint32_t dst_mod_id[kMaxDst];  // modulus id of each target (selects its twiddle table)
    // hats[t][i][k], k = 0..2: centred([(D / s_i) 2^(12 k)]_t) * 2^(-12 k), the factors that go with the three pieces
    // of a split source residue (split3; two pieces and 16 bits where every modulus is below 2^32).  Zero for padding sources.
    // The fused vector kernel (cut_source) uses [0], [1] and [3] = [2] * 2^24; with two pieces [0] and [3] = [1] * 2^16.
    double hats[kMaxDst][kMaxSrc][4];
    // centred(-0x80808080 sum_i [D / s_i]_t), which takes the constant out of the sum
    double dst_start[kMaxDst];
    // Matrix-core form (int8 MFMA, see ks_bconv_mfma.hip).  A source residue y = sum_a d_a 256^a is cut into five signed
    // digits; for every digit position a the factor F_a = centred([(D / s_i) 256^a]_t) is cut the same way into digits
    // e_b, so that y (D / s_i) = sum_b 256^b sum_a d_a e_{a,b} (mod t): five small integer sums per target, each a dot
    // product over (source, a) that the matrix cores accumulate exactly in 32 bits.
    // Each lane half reads mfma_t = mfma_sources(n) sources, every other one, and puts them into operand slots of
    // 16 bytes, up to three to a slot, slot = 2 * instruction + lane half; inside a slot, bytes 4 e + a (a < 4) belong to digit a of the slot's e-th source and byte 12 + e to its digit 4.
    // afac[t][b][slot] is the A-operand row of target t, digit plane b, in that byte order (zero where a slot has no source).
    uint32_t mfma_t;
    uint32_t mfma_src_limb[kMfmaSlots * 3];     // limb of the e-th source of a slot at 3 slot + e (padding: the first source's limb)
    alignas(16) int8_t afac[kMaxDst][kMfmaPlanes][kMfmaSlots][16];
    // everything the matrix-core kernel needs to know about a target, in one 32-byte record (one load per lane)
    struct alignas(32) TargetRec {
        Mod m;
        uint32_t mod_id, limb, pad[2];
    } trec[kMaxDst];
};

// The part of a plan a kernel launch carries by value in its arguments (no dependent load before the first source
// read): target count and source limbs in operand-slot order.
struct PlanMeta {
    uint32_t n_dst;
    uint32_t src_limb[kMfmaSlots * 3];
};
struct LaunchMeta {
    PlanMeta plan[kMaxDigits];
};
// The plans of one conversion launch (one per digit for ModUp, a single one otherwise): device copies plus the host
// facts the launchers need.
struct PlanSet {
    BConvPlan* d_plans = nullptr;  // [n_plans] device
    uint32_t n_plans = 0;
    uint32_t max_targets = 0;      // largest target count of a plan
    uint32_t shape_src = 0;        // source count the matrix-core operand slots were laid out for (the largest of the plans)
    uint32_t targets = 0, sixes = 0, products = 0;  // sums over the plans: targets, groups of six targets, sources x targets
    LaunchMeta meta{};
};

// Targets that a workgroup of the vector conversion takes: fewer targets = more workgroups and a shorter chain in each, but more re-reads
// and re-cuts of the sources.  Key-switches of random shapes, one and two targets against three by workgroups of one target: below 256
// -13 and -6 %, 512 to 1024 -4 and -3, 1024 to 2048 +0.2 and -1.9, 4096 to 8192 +6 and 0, above +10 and +2, four there -0.2.
//   Digits of different sizes have different numbers of targets: the workgroups counted are those that have work, not the digits times
// the largest number (110 key-switches on whose ModUp the two counts disagree: 0.2 to 4.4 % less time, 28 bits 8 / 8 / 1 -> 24 79.3 -> 76.8 us).
inline int vector_conversion_targets(const PlanSet& plans, uint32_t tiles, uint32_t n_polys) {
    const uint64_t ones = (uint64_t)tiles * plans.targets * n_polys;
    return ones <= 1024 ? 1 : ones <= 8192 ? 2 : 4;
}

// Everything the key-switching pipeline needs at one level ell.
struct Level {
    uint32_t ell = 0, ndig = 0, E = 0;     // E = ell + K extended limb count
    uint32_t n_new = 0;                    // sum over digits of (E - alpha_j): limbs produced by ModUp
    PlanSet modup;                         // one plan per digit
    PlanSet moddown;
    LimbMap lifted_map;                    // new limbs inside the [ndig][E][N] lifted bundle
    LimbMap special_map;                   // the K special limbs inside an [E][N] accumulator
    LimbMap q_map;                         // limbs 0..ell-1, modulus id = limb index
    uint32_t digit_lo[kMaxDigits], digit_hi[kMaxDigits];
    double* d_qlinv = nullptr;             // [ell-1] device: q_{ell-1}^-1 mod q_i (rescale)
    double* d_modup_scale = nullptr;       // [ell] device: N^-1 (D_j / q_i)^-1 mod q_i, j = digit of limb i
    // Division by P followed by the rescale (ell >= 2), both in one conversion to q_0..q_{ell-2} with limb ell-1 as a further
    // source.  merged: ModDown and rescale merged, a conversion from the basis {p_0..p_{K-1}, q_{ell-1}} (product D = P q_{ell-1}).
    // rescale: the sum of the conversion P -> q_i and P times the centred remainder of the dropped limb.
    PlanSet merged;                        // d_plans == nullptr when unavailable (K + 1 sources exceed kMaxLimbsIn)
    PlanSet rescale;
    LimbMap drop_map;                      // the K special limbs and limb ell-1 inside an [E][N] accumulator
    double* d_merged_scale = nullptr;      // [K+1] device: N^-1 (D / s)^-1 mod s, s in drop_map order
    double* d_rescale_scale = nullptr;     // [K+1] device: N^-1 (P / p_k)^-1 mod p_k, then N^-1 P^-1 mod q_{ell-1}
    double* d_pinv_last = nullptr;         // [K] device: p_k^-1 mod q_{ell-1}
    double* d_Dinv = nullptr;              // [ell-1] device: D^-1 mod q_i
    double Pmod_last = 0.0;                // P mod q_{ell-1}
};

}  // namespace ks

struct ks_ctx {
    int device = 0;
    uint32_t logN = 0, N = 0, L = 0, K = 0, dnum = 0, alpha = 0, M = 0;
    std::vector<uint64_t> mod, psi;       // host copies, index = modulus id
    ks::Mod* d_mod = nullptr;             // [M]
    double* d_ninv = nullptr;             // [M]  N^-1 mod m
    double* d_Pinv = nullptr;             // [L]  P^-1 mod q_i
    double* d_Pmod = nullptr;             // [L]  P mod q_i
    double* d_moddown_scale = nullptr;    // [K]  N^-1 (P / p_k)^-1 mod p_k
    double* d_tw_fwd = nullptr;           // [M][N] psi^brv(k)
    double* d_tw_inv = nullptr;           // [M][N] psi^-brv(k)
    double* d_trow = nullptr;             // [2][M][N/16] compact last-pass generators, forward then inverse
    double* d_w16 = nullptr;              // [2][M][8] powers of the primitive 16th root, forward then inverse
    ks::TwTables tw_fwd{}, tw_inv{};      // the three tables of each direction bundled for the row kernels
    std::vector<ks::Level> levels;        // index ell-1
    int opt[KS_OPT_COUNT_] = {};          // ks_ctx_set_option values, index = option id
    int pieces = 3;                       // pieces a source residue is cut into by the fused conversion: 2 iff every modulus < 2^32
    mutable std::mutex mu;
    mutable std::map<std::vector<uint32_t>, ks::PlanSet> bconv_cache;  // key: n_src, src ids, dst ids
};

namespace ks {

// ---- host number theory (ks_ctx.hip) ----
uint64_t h_mulmod(uint64_t a, uint64_t b, uint64_t m);
uint64_t h_powmod(uint64_t a, uint64_t e, uint64_t m);
uint64_t h_invmod(uint64_t a, uint64_t m);
// shape_src: the source count that fixes the operand-slot layout of the matrix-core tables (all plans of one launch must
// agree on it); 0 = n_src.  The last n_extra sources are not part of the basis: their factor is the product of all moduli
// of the others, which they do not enter.
void fill_bconv_plan(const ks_ctx* c, BConvPlan* plan, const uint32_t* src_ids, const uint16_t* src_limb, uint32_t n_src,
                     const uint32_t* dst_ids, const uint16_t* dst_limb, uint32_t n_dst, uint32_t shape_src = 0, uint32_t n_extra = 0);

// thread-local HIP error text
void set_hip_error(hipError_t e, const char* where);

// Optional per-kernel timing (ks_profile_enable): when on, every launcher brackets its kernel with a pair of
// HIP events on the launch stream and books the kernel's algorithmic bytes (what it must read plus write).
struct ProfScope {
    // ops: algorithmic fp64 vector instructions per lane (FMA, MUL, ADD and RNDNE each count one)
    ProfScope(const char* name, double bytes, hipStream_t s, double ops = 0.0);
    ~ProfScope();
    int slot;
    hipStream_t stream;
};

// Dispatch on the ring degree: N = 2^12 .. 2^16 <-> R = N / 256 = 2^4 .. 2^8 rows.
#define KS_FOR_LOG_R(logN, M) \
    switch (logN) {           \
        case 12: M(4); break; \
        case 13: M(5); break; \
        case 14: M(6); break; \
        case 15: M(7); break; \
        default: M(8); break; \
    }

// ---- launchers: all asynchronous on `s`, no allocation ----
// Both directions on limbs of 64-bit words, in place: coefficients <-> evaluations, canonical residues in and out.
void launch_ntt(const ks_ctx* c, const LimbMap& map, uint64_t* data, uint64_t ps_words, uint32_t n_polys, bool inverse, hipStream_t s);
// both directions on limbs in 32-bit words, in place (canonical residues between the two passes as well)
void launch_ntt_u32(const ks_ctx* c, const LimbMap& map, uint32_t* data, uint64_t ps_words, uint32_t n_polys, bool inverse,
                    hipStream_t s);
// The inverse transform that feeds a conversion (packed limbs: ks_tiles.hpp).  Rows: `in` holds words of in_word = 8 or 4 bytes, or
// (1) packed accumulators, converted in place; in_ps counts words (bytes for 1), out_ps bytes.
void launch_inv_rows_packed(const ks_ctx* c, const LimbMap& map, const void* in, uint64_t in_ps, int in_word, uint8_t* out, uint64_t out_ps,
                            uint32_t n_polys, hipStream_t s);
// Columns, in place: leaves the conversion's sources.  scale_tab: multiplier applied with the final reduction, by position in `map`.
void launch_inv_cols_packed(const ks_ctx* c, const LimbMap& map, uint8_t* data, uint64_t ps_bytes, uint32_t n_polys, const double* scale_tab,
                            hipStream_t s);

// The kernel of both conversions of a call (ks_fused.hip): 0 vector, 8 or 16 matrix cores with tiles of that many columns.
int conversion_tile(const ks_ctx* c, const PlanSet& up, uint32_t up_polys, const PlanSet& down, uint32_t down_polys);
// Fused base conversion + column half of the forward transform, with the kernel `tile` (conversion_tile).  y: packed sources
// y_i = [x_i N^-1 (D/s_i)^-1]; out: packed limbs ready for the row half; strides in bytes.  One plan per blockIdx.y group.
void launch_bconv_ntt_cols(const ks_ctx* c, const PlanSet& plans, uint32_t limbs_moved_per_poly, const uint8_t* y, uint64_t y_ps,
                           uint8_t* out, uint64_t out_ps, uint32_t n_polys, int tile, hipStream_t s);
// The same conversion + column half on the matrix cores (ks_bconv_mfma.hip); tl = targets per lane half, 1..3.
void launch_bconv_mfma_ntt_cols(const ks_ctx* c, const PlanSet& plans, const uint8_t* y, uint64_t y_ps, uint8_t* out,
                                uint64_t out_ps, uint32_t n_polys, int tl, bool wide, hipStream_t s);
// Upload host plans as a PlanSet (allocates; ks_ctx_create and bconv plan registration only).  Returns a HIP error code.
hipError_t upload_plans(const BConvPlan* host_plans, uint32_t n_plans, uint32_t shape_src, PlanSet* out);
// Rotations handled by one launch of the gather kernels (more are chained).
constexpr int kMacRotations = 16;
struct MacRotations {
    uint32_t n;
    uint32_t galois[kMacRotations];
    const void* key[kMacRotations];  // [dnum][2][L+K][N], 64- or 32-bit words
    const void* pt[kMacRotations];   // [L+K][N], same word size as the keys
};
struct FinishRotations {
    uint32_t galois[kMacRotations];
};
// Fused row half of the forward transform of the raised digits + inner product with the key.
// d_word: bytes of a word of d, 8 or 4, or 1: packed limbs in rows order (then d_ps counts bytes); words32: the key holds one residue
// per 32-bit word (4-byte words of d imply them).  acc: [b][2][E] packed.  The ciphertext limbs are in rows order; the special limbs have been through the row half of their inverse
// transform and are in columns order.  drop_addend != nullptr: limb ell-1 joins the special limbs after P times limb ell-1 of that
// addend ([b][2][ell] packed) has been added.  dropped_only: only the limbs that the division drops, the special ones and that one.
void launch_rows_inner_product(const ks_ctx* c, const Level& lv, const void* d, uint64_t d_ps, const uint8_t* lifted,
                               const void* evk, uint8_t* acc, uint32_t batch, hipStream_t s, int d_word, bool words32,
                               const uint8_t* drop_addend, bool dropped_only);
// Whether a call forms the sums of the n_stay limbs that stay where the division ends (launch_rows_key_finish) instead of in memory.
bool sums_meet_division(const ks_ctx* c, const Level& lv, uint32_t n_stay, uint32_t batch);
// Fused row half of the forward transform of the converted limbs (conv, [b][2][ell] packed) + (acc - conv) P^-1 (+ addend);
// the ciphertext limbs of acc ([b][2][E] packed) are in rows order.
// fs == nullptr: multiply by P^-1, ell output limbs; with `rotations` (their galois elements are read) acc and conv hold that many
// batches one behind the other, whose outputs are out_rot_stride words apart, and the addend, in the word size of the output and
// addend_batch_stride words between batch items, is added to component 0 through sigma_galois.  Otherwise (division by P and a rescale): multiply by fs->mul[i], add the
// packed addend ([b][2][ell]) times fs->addend_mul[i], write the first fs->out_limbs limbs per component.
struct FinishScale {
    const double* mul;
    const double* addend_mul;
    uint32_t out_limbs;
};
void launch_rows_moddown_finish(const ks_ctx* c, const Level& lv, const uint8_t* acc, const uint8_t* conv, void* out,
                                uint64_t out_batch_stride, const void* addend, uint64_t addend_batch_stride,
                                const MacRotations* rotations, uint64_t out_rot_stride, uint32_t batch, hipStream_t s,
                                const FinishScale* fs = nullptr, bool out_words32 = false);
// The inner product on the limbs that stay and launch_rows_moddown_finish in one: out = (sum - conv) P^-1, or with fs (sum - conv) fs->mul[i] +
// addend fs->addend_mul[i].  out has the key's words.
void launch_rows_key_finish(const ks_ctx* c, const Level& lv, const void* d, uint64_t d_ps, const uint8_t* lifted, const void* evk,
                            const uint8_t* conv, const uint8_t* addend, void* out, uint64_t out_bs, uint32_t batch, hipStream_t s,
                            int d_word, bool words32, const FinishScale* fs);
// Remainder of the dropped limb for a rescale.  acc: [polys][E], the drop_map limbs as sources of a conversion (canonical: y_k on the
// special limbs, P^-1 times the dropped limb's sum on limb ell-1); limb ell-1 becomes the centred remainder of (sum - converted
// special part) P^-1 modulo q_{ell-1}, a signed source.
void launch_rescale_remainder(const ks_ctx* c, const Level& lv, uint8_t* acc, uint32_t n_polys, hipStream_t s);

// The standalone conversion (ks_bconv.hip: the choice of the kernel, and the vector kernel).
// words32: in and out hold one residue per 32-bit word (strides in words either way)
void launch_bconv(const ks_ctx* c, const PlanSet& plans, uint32_t limbs_moved_per_poly, const void* in, uint64_t in_poly_stride,
                  void* out, uint64_t out_poly_stride, uint32_t n_polys, hipStream_t s, bool words32);
// the same on the matrix cores (ks_bconv_mfma.hip)
void launch_bconv_mfma(const ks_ctx* c, const PlanSet& plans, uint32_t limbs_moved_per_poly, const void* in, uint64_t in_poly_stride,
                       void* out, uint64_t out_poly_stride, uint32_t n_polys, hipStream_t s, bool words32);

// What the sigma_g gathers of a rotation read, for a group of up to 8 ciphertexts: slabs of N slots, slab j E + pos the
// finished raised digit j at limb position pos (in the slots of a digit's own positions the limbs of the polynomial
// itself), slabs ndig E + pos, pos < ell, the limbs of the addend c0 where a caller asked for them.  A slot holds the
// residues of all `group` ciphertexts side by side, so that one gathered slot is one contiguous access or two for every
// ciphertext that needs it.  lo: the 32-bit low words, per 64 consecutive slots first the words of up to four ciphertexts, then
// those of the others (a wavefront reads both parts as whole lines); hi != nullptr: hi[slot] holds the bits above (moduli are
// below 2^36) as one 4-bit field per ciphertext in a word of gather_hi_bytes(group).  hi == nullptr: moduli below 2^32, lo alone.
//   The group is the batch, whatever it is.  Rounded up to 1, 2, 4 or 8, five ciphertexts were transformed, written and
// gathered as eight: one rotate-multiply-accumulate of five, N = 2^16, E = 32, three digits 504 us against 470 (28-bit moduli 447
// against 417); at N = 2^14 91 against 82.
//   c0 != nullptr: rotate_mac gathers the addend from these ciphertexts (64-bit words with a packed bundle, 32-bit words with
// a 32-bit one; c0_ps words apart) instead of from slabs of the bundle.
struct GatherBundle {
    uint32_t* lo;
    uint8_t* hi;
    uint32_t group;
    const void* c0;
    uint64_t c0_ps;
};
constexpr int kMaxGroup = 8;
constexpr uint32_t gather_hi_bytes(uint32_t group) { return group > 4 ? 4 : group > 2 ? 2 : 1; }
template <int G>
struct SlotLayout {
    static constexpr int FIRST = G < 4 ? G : 4, REST = G - FIRST;  // low words of a slot in the first and in the second part
    using HW = std::conditional_t<gather_hi_bytes(G) == 4, uint32_t, std::conditional_t<gather_hi_bytes(G) == 2, uint16_t, uint8_t>>;
};
// One launch of a kernel with the group size as a template parameter: LAUNCH(G)
#define KS_FOR_GROUP(group, LAUNCH)   \
    switch (group) {                  \
        case 1: LAUNCH(1); break;     \
        case 2: LAUNCH(2); break;     \
        case 3: LAUNCH(3); break;     \
        case 4: LAUNCH(4); break;     \
        case 5: LAUNCH(5); break;     \
        case 6: LAUNCH(6); break;     \
        case 7: LAUNCH(7); break;     \
        default: LAUNCH(8); break;    \
    }
// Fill a bundle in one launch.  raised: the row half of the forward transform of the raised limbs (`lifted`,
// [b][ndig][E] packed limbs after the column half), all digits.  The polynomials' own limbs d[b][pos] and, c0 != nullptr,
// the addend's limbs c0[b][pos] (64-bit words with a packed bundle, 32-bit words with a 32-bit one; ps words apart) are
// copied.
void launch_gather_bundle_rows(const ks_ctx* c, const Level& lv, const uint8_t* lifted, const void* d, const void* c0, uint64_t ps,
                               const GatherBundle& out, bool raised, hipStream_t s);

// acc[r][b][c][pos] = sum_j sigma_{g_r}(src_j)[pos] * key_r[j][c][ext_id(pos)] for every rotation r of `rot` (pt unused);
// src_j[pos] = slab j E + pos of the bundle.
// key_words32: keys (and plaintexts) hold one residue per 32-bit word; 32-bit sources imply 32-bit keys.
// acc: [r][b][2][E], packed limbs in rows order.
// special_only: only the limbs that the division drops.
void launch_inner_product(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, uint8_t* acc, hipStream_t s,
                          bool key_words32, bool special_only);

// Whether a group of rotations of `group` ciphertexts forms the sums of the ciphertext limbs where the division ends (launch_rotate_finish)
// instead of in memory.
bool rotations_meet_division(const ks_ctx* c, const Level& lv, uint32_t group, uint32_t n_rot);
// launch_inner_product on the ciphertext limbs and launch_rows_moddown_finish with rotations in one; conv: [r][b][2][ell] packed.
// out: [b][r][2][ell] words, batch items out_bs apart; c0: [b][2][ell] words.
void launch_rotate_finish(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, const uint8_t* conv, void* out,
                          uint64_t out_bs, const void* c0, hipStream_t s, bool words32);

// u[b][c][pos] (+)= sum_r pt_r[pos] * (sum_j sigma_r(src_j)[pos] key_r[j][c][pos] + [c = 0][pos < ell] P sigma_r(c0)[pos]);
// src: c1 and its finished raised digits, and c0.  u: packed limbs in rows order.  accumulate: add to what u already holds.
// galois[r] == 1: the term is P (c0, c1) and key[r] is not read; pt[r] == nullptr: the constant 1.
void launch_rotate_mac(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, uint8_t* u,
                       bool accumulate, hipStream_t s, bool key_words32 = false);

// The sums of several rows of diagonals over the same rotations in one launch: u_i (+)= sum_r pt[i][r] * (...) as above, i < n (2 or
// kMacRows), u_i u_stride bytes apart.  The bundle holds c0.
constexpr uint32_t kMacRows = 4;
struct MacRows {
    uint32_t n;
    const void* pt[kMacRows][kMacRotations];
};
void launch_rotate_mac_rows(const ks_ctx* c, const Level& lv, const GatherBundle& src, const MacRotations& rot, const MacRows& rows, uint8_t* u,
                            uint64_t u_stride, bool accumulate, hipStream_t s, bool key_words32);

// The key-switch chain behind ks_keyswitch / ks_keyswitch_u32 (argument checks included); ws is any device buffer of
// at least ks_workspace_bytes(KS_OP_KEYSWITCH) bytes, whose contents need no initialisation.
int keyswitch_impl(const ks_ctx* c, const void* d, uint32_t ell, const void* evk, void* out, uint32_t batch, void* ws,
                   size_t ws_bytes, void* stream, bool words32);

// Resolve this device's copy of the library-owned static scratch array (ks_static.hip); called by ks_ctx_create with
// the device current.  Returns a HIP error code.
hipError_t bind_static_scratch(int device);

// Tensor product of two ciphertexts ([batch][2][ell][N] words): d0 = b1 b2, d1 = a1 b2 + a2 b1 -> dq [batch][2][ell], d2 = a1 a2 ->
// d2 [batch][ell], packed limbs in rows order; the row half of d2's inverse transform -> inv [batch][ell] in columns order.
void launch_tensor_inv_rows(const ks_ctx* c, const void* cta, const void* ctb, uint32_t ell, uint8_t* dq, uint8_t* d2, uint8_t* inv,
                            uint32_t batch, hipStream_t s, bool in_words32);
}  // namespace ks
