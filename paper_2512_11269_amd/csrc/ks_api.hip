// The extern "C" entry points: argument checks, workspace carving and the kernel chains.
#include <algorithm>

#include "ks_internal.hpp"

using namespace ks;

namespace {

// Ciphertexts that the workspace of a pipeline is sized for; more are processed in passes (rotations of eight, the group of a gather;
// key-switches and multiplications: ciphertexts_at_a_time).
constexpr uint32_t kChunk = 8;
static_assert(kChunk <= kMaxGroup, "ciphertexts of one gather bundle");
constexpr uint32_t kRotGroup = 4;  // hoisted rotations that the workspace is sized for; a group of a gather launch

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int finish(const char* where) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_hip_error(e, where);
        return KS_EHIP;
    }
    return KS_OK;
}

// Bytes of the packed regions of a chunk of `bc` ciphertexts.
struct KsWorkspace {
    uint64_t coeff, lifted, acc, conv;   // [bc][ell], [bc][ndig][E], [bc][2][E], [bc][2][ell] packed limbs
};

KsWorkspace ks_ws_regions(const ks_ctx* c, const Level& lv, uint32_t bc) {
    const uint64_t limb = packed_limb_bytes(c->N);
    KsWorkspace w;
    w.coeff = (uint64_t)bc * lv.ell * limb;
    w.lifted = (uint64_t)bc * lv.ndig * lv.E * limb;
    w.acc = (uint64_t)bc * 2 * lv.E * limb;
    w.conv = (uint64_t)bc * 2 * lv.ell * limb;
    return w;
}

// What ks_workspace_bytes asks for: the same regions with 8 bytes a residue and a packed copy of the ciphertext limbs of the
// accumulators, in 64-bit words.  More than ks_ws_regions adds up to, and kept: the figure is part of the interface.
struct KsWorkspaceWords {
    uint64_t coeff, lifted, acc, conv, accq;
    uint64_t total() const { return coeff + lifted + acc + conv + accq; }
};

KsWorkspaceWords ks_ws_words(const ks_ctx* c, const Level& lv, uint32_t bc) {
    const uint64_t N = c->N;
    KsWorkspaceWords w;
    w.coeff = (uint64_t)bc * lv.ell * N;
    w.lifted = (uint64_t)bc * lv.ndig * lv.E * N;
    w.acc = (uint64_t)bc * 2 * lv.E * N;
    w.conv = (uint64_t)bc * 2 * lv.ell * N;
    w.accq = packed_limb_bytes(w.conv) / 8;
    return w;
}

// mod_up from the row half of the inverse transform on: coeff [bc][ell] packed.
void mod_up_from_rows(const ks_ctx* c, const Level& lv, uint8_t* coeff, uint8_t* lifted, uint32_t bc, int tile, hipStream_t s) {
    const uint64_t limb = packed_limb_bytes(c->N), coeff_ps = lv.ell * limb, lifted_ps = (uint64_t)lv.ndig * lv.E * limb;
    // the column half also multiplies by N^-1 (D_j/q_i)^-1 and leaves the sources of the conversion
    launch_inv_cols_packed(c, lv.q_map, coeff, coeff_ps, bc, lv.d_modup_scale, s);
    launch_bconv_ntt_cols(c, lv.modup, lv.ell + lv.n_new, coeff, coeff_ps, lifted, lifted_ps, bc, tile, s);
}

// Decompose and raise: d (evaluation domain, `bc` polynomials d_ps words apart) -> lifted [bc][ndig][E] packed.
// The raised limbs stop after the column half of the forward transform; the row half is left to the
// fused inner product, or to mod_up_for_gather below.  tile: the conversion kernel of the call (conversion_tile).
void mod_up(const ks_ctx* c, const Level& lv, const void* d, uint64_t d_ps, uint8_t* coeff, uint8_t* lifted, uint32_t bc,
            int tile, hipStream_t s, bool d_words32 = false) {
    launch_inv_rows_packed(c, lv.q_map, d, d_ps, d_words32 ? 4 : 8, coeff, lv.ell * packed_limb_bytes(c->N), bc, s);
    mod_up_from_rows(c, lv, coeff, lifted, bc, tile, s);
}

// Words of workspace the bundle of a chunk of bc ciphertexts takes: low words, then (64-bit operands) the bits above;
// with_c0: the addend's limbs as well.
static uint64_t gather_lo_words(const ks_ctx* c, const Level& lv, uint32_t bc, bool with_c0) {
    return ((uint64_t)lv.ndig * lv.E + (with_c0 ? lv.ell : 0)) * c->N * bc / 2;
}
static uint64_t gather_words(const ks_ctx* c, const Level& lv, uint32_t bc, bool with_c0, bool words32) {
    const uint64_t slots = ((uint64_t)lv.ndig * lv.E + (with_c0 ? lv.ell : 0)) * c->N;
    return gather_lo_words(c, lv, bc, with_c0) + (words32 ? 0 : slots * gather_hi_bytes(bc) / 8);
}

// Rotations from which on the bundle holds the addend c0; below, copying it there costs more than gathering it from the
// ciphertexts (24 limbs of 100, written and read back).  Rotate-multiply-accumulate, N = 2^16, E = 32, three digits, copied -> gathered:
// one rotation of 1, 3 and 8 ciphertexts 131 -> 128, 293 -> 282 and 688 -> 665 us (28-bit moduli 117 -> 116, 261 -> 253,
// 622 -> 607); five -3.2, -2.1 and -0.5 %; six -2.4, -1.9 and +0.6 %; sixteen +0.2, +0.1 and +3.7 %.
constexpr uint32_t kC0InBundle = 6;

// mod_up finished for the rotation gathers: `region` (gather_words() 64-bit words) ends as the bundle they read.  `lifted` is only
// scratch here.  raised == false: only the own limbs (and c0) are filled in, for a caller whose rotations are all identities.
// n_rot: rotations that read the bundle.
static GatherBundle mod_up_for_gather(const ks_ctx* c, const Level& lv, const void* d, const void* c0, uint64_t d_ps, uint8_t* coeff,
                                      uint8_t* lifted, uint64_t* region, uint32_t bc, uint32_t n_rot, int tile, hipStream_t s, bool words32,
                                      bool raised = true) {
    if (raised) mod_up(c, lv, d, d_ps, coeff, lifted, bc, tile, s, words32);
    const bool with_c0 = c0 && n_rot >= kC0InBundle;
    const GatherBundle bundle{reinterpret_cast<uint32_t*>(region),
                              words32 ? nullptr : reinterpret_cast<uint8_t*>(region + gather_lo_words(c, lv, bc, with_c0)),
                              bc, with_c0 ? nullptr : c0, d_ps};
    launch_gather_bundle_rows(c, lv, lifted, d, with_c0 ? c0 : nullptr, d_ps, bundle, raised, s);
    return bundle;
}

// Inner product of the raised digits of d with the key, and the division of both sums: by P, or (addend: [b][2][ell] packed) of the sums +
// P addend by P q_{ell-1} in one conversion to q_0..q_{ell-2}, limb ell-1 joining the special limbs as a source.  merged: ModDown and
// rescale merged (floor throughout); otherwise floor(/ P), then round(/ q_{ell-1}).  The inner product has already added the dropped
// limb's addend and run the row half of the inverse transform on the sources.
void key_sums_and_division(const ks_ctx* c, const Level& lv, const void* d, uint64_t d_ps, const uint8_t* lifted, const void* evk, uint8_t* acc,
                           uint8_t* conv, void* out, uint64_t out_bs, uint32_t bc, int tile, hipStream_t s, int d_word, bool words32,
                           const uint8_t* addend, bool merged) {
    const uint64_t limb = packed_limb_bytes(c->N), acc_ps = lv.E * limb, conv_ps = lv.ell * limb;
    const bool meet = sums_meet_division(c, lv, addend ? lv.ell - 1 : lv.ell, bc);
    launch_rows_inner_product(c, lv, d, d_ps, lifted, evk, acc, bc, s, d_word, words32, addend, meet);
    launch_inv_cols_packed(c, addend ? lv.drop_map : lv.special_map, acc, acc_ps, 2 * bc,
                           !addend ? c->d_moddown_scale : merged ? lv.d_merged_scale : lv.d_rescale_scale, s);
    if (addend && !merged) launch_rescale_remainder(c, lv, acc, 2 * bc, s);
    // K sources and ell targets, or one target less and one source more
    launch_bconv_ntt_cols(c, !addend ? lv.moddown : merged ? lv.merged : lv.rescale, c->K + lv.ell, acc, acc_ps, conv, conv_ps, 2 * bc, tile, s);
    const FinishScale fs{lv.d_Dinv, lv.d_qlinv, lv.ell - 1};
    if (meet) launch_rows_key_finish(c, lv, d, d_ps, lifted, evk, conv, addend, out, out_bs, bc, s, d_word, words32, addend ? &fs : nullptr);
    else launch_rows_moddown_finish(c, lv, acc, conv, out, out_bs, addend, 0, nullptr, 0, bc, s, addend ? &fs : nullptr, words32);
}

// Division by P of both accumulators: INTT of the special limbs (in place), fused base conversion + column half, fused row
// half + (acc - conv) P^-1.
void mod_down(const ks_ctx* c, const Level& lv, uint8_t* acc, uint8_t* conv, void* out, uint64_t out_bs,
              uint32_t bc, int tile, hipStream_t s, bool out_words32 = false) {
    const uint64_t limb = packed_limb_bytes(c->N), acc_ps = lv.E * limb, conv_ps = lv.ell * limb;
    launch_inv_rows_packed(c, lv.special_map, acc, acc_ps, 1, acc, acc_ps, 2 * bc, s);
    launch_inv_cols_packed(c, lv.special_map, acc, acc_ps, 2 * bc, c->d_moddown_scale, s);
    launch_bconv_ntt_cols(c, lv.moddown, c->K + lv.ell, acc, acc_ps, conv, conv_ps, 2 * bc, tile, s);
    launch_rows_moddown_finish(c, lv, acc, conv, out, out_bs, nullptr, 0, nullptr, 0, bc, s, nullptr, out_words32);
}

}  // namespace

extern "C" size_t ks_workspace_bytes(const ks_ctx* c, int op, uint32_t ell, uint32_t batch, uint32_t n_rot) {
    if (!c || c->K == 0 || ell < 1 || ell > c->L || batch == 0) return 0;
    const Level& lv = c->levels[ell - 1];
    const uint32_t bc = std::min(batch, kChunk);
    const uint64_t N = c->N;
    uint64_t words = ks_ws_words(c, lv, bc).total();
    switch (op) {
        case KS_OP_KEYSWITCH: break;
        case KS_OP_ROTATE_HOISTED:
        case KS_OP_ROTATE_HOISTED_U32:
            if (n_rot == 0) return 0;
            // the gathers' sources (rotate-multiply-accumulate may keep c0 among them)
            words += gather_words(c, lv, bc, n_rot >= kC0InBundle, op == KS_OP_ROTATE_HOISTED_U32);
            // accumulators and converted limbs for a whole group of rotations; the ciphertext limbs of a group's accumulators, packed
            words += (uint64_t)(std::min(n_rot, kRotGroup) - 1) * bc * (2 * lv.E + 2 * ell) * N;
            words += (uint64_t)(std::min(n_rot, kRotGroup) - 1) * ks_ws_words(c, lv, bc).accq;
            break;
        case KS_OP_BSGS:
        case KS_OP_BSGS_U32: {
            // accumulators of the outer level, inner result [bc][2][ell], the gathers' sources of both levels (the
            // inner results are 64-bit words either way)
            const KsWorkspaceWords w = ks_ws_words(c, lv, bc);
            words += w.acc + (uint64_t)bc * 2 * ell * N + gather_words(c, lv, bc, true, op == KS_OP_BSGS_U32) +
                     gather_words(c, lv, bc, false, false);
            break;
        }
        case KS_OP_HMULT_RELIN_RESCALE:
            if (ell < 2) return 0;
            // d2 [bc][ell], (d0, d1) packed like the accumulator limbs
            words += (uint64_t)bc * ell * N + ks_ws_words(c, lv, bc).accq;
            break;
        default: return 0;
    }
    return (size_t)words * sizeof(uint64_t);
}

// Ciphertexts that a key-switch or multiplication takes at a time, given the bytes one of them takes: kChunk, or as many as the
// workspace holds (a caller brings what ks_workspace_bytes asks for, 8 bytes a residue; the packed regions of thirteen or fourteen fit) where
// that makes fewer passes, evenly filled.  Key-switches in passes of eight -> so many: N = 2^12, 12 ciphertexts 79 -> 45 us, 64 327 -> 224;
// N = 2^14 185 -> 151 and 918 -> 841; N = 2^16, L = 24 803 -> 753 and 4014 -> 3887; multiplications at L = 35, 64 of them 7086 -> 7046.
// As many passes as before stay as they are (seven and seven for eight and six was up to 12 % slower).
static uint32_t ciphertexts_at_a_time(const ks_ctx* c, const Level& lv, int op, uint32_t batch, uint64_t bytes_of_one) {
    if (batch <= kChunk) return batch;
    const uint32_t fit = (uint32_t)(ks_workspace_bytes(c, op, lv.ell, batch, 0) / bytes_of_one), passes = (batch + fit - 1) / fit;
    return passes == (batch + kChunk - 1) / kChunk ? kChunk : (batch + passes - 1) / passes;
}

static int check_map_args(const ks_ctx* c, const void* data, const uint32_t* mod_ids, uint32_t nlimbs, LimbMap* map) {
    if (!c || !data || !mod_ids || nlimbs == 0 || nlimbs > (uint32_t)kMaxLimbs || !aligned16(data)) return KS_EINVAL;
    map->n = nlimbs;
    for (uint32_t i = 0; i < nlimbs; ++i) {
        if (mod_ids[i] >= c->M) return KS_EINVAL;
        map->off[i] = (uint16_t)i;
        map->mod[i] = (uint8_t)mod_ids[i];
    }
    return KS_OK;
}

extern "C" int ntt_fwd(const ks_ctx* c, uint64_t* data, const uint32_t* mod_ids, uint32_t nlimbs, uint32_t batch, void* stream) {
    LimbMap map;
    int rc = check_map_args(c, data, mod_ids, nlimbs, &map);
    if (rc != KS_OK) return rc;
    if (batch == 0) return KS_OK;
    if ((uint64_t)batch * nlimbs > (1u << 26)) return KS_EINVAL;
    const uint64_t ps = (uint64_t)nlimbs * c->N;
    launch_ntt(c, map, data, ps, batch, false, static_cast<hipStream_t>(stream));
    return finish("ntt_fwd");
}

extern "C" int ntt_inv(const ks_ctx* c, uint64_t* data, const uint32_t* mod_ids, uint32_t nlimbs, uint32_t batch, void* stream) {
    LimbMap map;
    int rc = check_map_args(c, data, mod_ids, nlimbs, &map);
    if (rc != KS_OK) return rc;
    if (batch == 0) return KS_OK;
    if ((uint64_t)batch * nlimbs > (1u << 26)) return KS_EINVAL;
    const uint64_t ps = (uint64_t)nlimbs * c->N;
    launch_ntt(c, map, data, ps, batch, true, static_cast<hipStream_t>(stream));
    return finish("ntt_inv");
}

static bool moduli_fit_u32(const ks_ctx* c) {
    for (uint64_t m : c->mod)
        if (m >> 32) return false;
    return true;
}

static int ntt_u32(const ks_ctx* c, uint32_t* data, const uint32_t* mod_ids, uint32_t nlimbs, uint32_t batch, void* stream,
                   bool inverse) {
    LimbMap map;
    int rc = check_map_args(c, data, mod_ids, nlimbs, &map);
    if (rc != KS_OK) return rc;
    if (!moduli_fit_u32(c)) return KS_EINVAL;
    if (batch == 0) return KS_OK;
    if ((uint64_t)batch * nlimbs > (1u << 26)) return KS_EINVAL;
    launch_ntt_u32(c, map, data, (uint64_t)nlimbs * c->N, batch, inverse, static_cast<hipStream_t>(stream));
    return finish(inverse ? "ntt_inv_u32" : "ntt_fwd_u32");
}

extern "C" int ntt_fwd_u32(const ks_ctx* c, uint32_t* data, const uint32_t* mod_ids, uint32_t nlimbs, uint32_t batch, void* stream) {
    return ntt_u32(c, data, mod_ids, nlimbs, batch, stream, false);
}

extern "C" int ntt_inv_u32(const ks_ctx* c, uint32_t* data, const uint32_t* mod_ids, uint32_t nlimbs, uint32_t batch, void* stream) {
    return ntt_u32(c, data, mod_ids, nlimbs, batch, stream, true);
}

// Key of a registered conversion: n_src, source ids, target ids.  Returns KS_OK or KS_EINVAL.
static int bconv_key(const ks_ctx* c, const uint32_t* src_ids, uint32_t n_src, const uint32_t* dst_ids, uint32_t n_dst,
                     std::vector<uint32_t>* key) {
    if (!c || !src_ids || !dst_ids) return KS_EINVAL;
    if (n_src == 0 || n_src > (uint32_t)kMaxLimbsIn || n_dst == 0 || n_dst > 255) return KS_EINVAL;
    key->push_back(n_src);
    for (uint32_t i = 0; i < n_src; ++i) {
        if (src_ids[i] >= c->M) return KS_EINVAL;
        for (uint32_t k = 0; k < i; ++k)
            if (src_ids[k] == src_ids[i]) return KS_EINVAL;
        key->push_back(src_ids[i]);
    }
    for (uint32_t t = 0; t < n_dst; ++t) {
        if (dst_ids[t] >= c->M) return KS_EINVAL;
        key->push_back(dst_ids[t]);
    }
    return KS_OK;
}

extern "C" int bconv_prepare(ks_ctx* c, const uint32_t* src_ids, uint32_t n_src, const uint32_t* dst_ids, uint32_t n_dst) {
    std::vector<uint32_t> key;
    int rc = bconv_key(c, src_ids, n_src, dst_ids, n_dst, &key);
    if (rc != KS_OK) return rc;
    std::lock_guard<std::mutex> lock(c->mu);
    if (c->bconv_cache.count(key)) return KS_OK;
    if (hipSetDevice(c->device) != hipSuccess) return KS_EHIP;
    std::vector<BConvPlan> plan(1);
    uint16_t src_limb[kMaxSrc];
    std::vector<uint16_t> dst_limb(n_dst);
    for (uint32_t i = 0; i < n_src; ++i) src_limb[i] = (uint16_t)i;
    for (uint32_t t = 0; t < n_dst; ++t) dst_limb[t] = (uint16_t)t;
    fill_bconv_plan(c, plan.data(), src_ids, src_limb, n_src, dst_ids, dst_limb.data(), n_dst);
    PlanSet set;
    hipError_t e = upload_plans(plan.data(), 1, n_src, &set);
    if (e != hipSuccess) {
        set_hip_error(e, "bconv_prepare: table upload");
        return KS_EHIP;
    }
    c->bconv_cache[key] = set;
    return KS_OK;
}

static int bconv_impl(const ks_ctx* c, const void* in, const uint32_t* src_ids, uint32_t n_src, void* out, const uint32_t* dst_ids,
                      uint32_t n_dst, uint32_t batch, void* stream, bool words32) {
    if (!in || !out || !aligned16(in) || !aligned16(out)) return KS_EINVAL;
    std::vector<uint32_t> key;
    int rc = bconv_key(c, src_ids, n_src, dst_ids, n_dst, &key);
    if (rc != KS_OK) return rc;
    if (words32 && !moduli_fit_u32(c)) return KS_EINVAL;
    PlanSet set;
    {
        std::lock_guard<std::mutex> lock(c->mu);
        auto it = c->bconv_cache.find(key);
        if (it == c->bconv_cache.end()) return KS_ENOTPREPARED;  // compute calls never allocate: register with bconv_prepare
        set = it->second;
    }
    if (batch == 0) return KS_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint64_t N = c->N, word = words32 ? 4 : 8;
    for (uint32_t b0 = 0; b0 < batch; b0 += 32768) {
        const uint32_t nb = std::min(batch - b0, 32768u);
        const char* ip = static_cast<const char*>(in) + (uint64_t)b0 * n_src * N * word;
        char* op = static_cast<char*>(out) + (uint64_t)b0 * n_dst * N * word;
        launch_bconv(c, set, n_src + n_dst, ip, (uint64_t)n_src * N, op, (uint64_t)n_dst * N, nb, s, words32);
    }
    return finish(words32 ? "bconv_u32" : "bconv");
}

extern "C" int bconv(const ks_ctx* c, const uint64_t* in, const uint32_t* src_ids, uint32_t n_src, uint64_t* out,
                     const uint32_t* dst_ids, uint32_t n_dst, uint32_t batch, void* stream) {
    return bconv_impl(c, in, src_ids, n_src, out, dst_ids, n_dst, batch, stream, false);
}

extern "C" int bconv_u32(const ks_ctx* c, const uint32_t* in, const uint32_t* src_ids, uint32_t n_src, uint32_t* out,
                         const uint32_t* dst_ids, uint32_t n_dst, uint32_t batch, void* stream) {
    return bconv_impl(c, in, src_ids, n_src, out, dst_ids, n_dst, batch, stream, true);
}

static int check_pipeline_args(const ks_ctx* c, uint32_t ell, uint32_t min_ell, const void* a, const void* b, const void* o,
                               const void* ws) {
    if (!c || c->K == 0 || !a || !b || !o || !aligned16(a) || !aligned16(b) || !aligned16(o)) return KS_EINVAL;
    if (ell < min_ell || ell > c->L) return KS_EINVAL;
    if (!ws || !aligned16(ws)) return KS_EWORKSPACE;
    return KS_OK;
}

// d, evk and out in 64-bit words, or all three in 32-bit words (words32; every modulus then below 2^32).
int ks::keyswitch_impl(const ks_ctx* c, const void* d, uint32_t ell, const void* evk, void* out, uint32_t batch, void* ws,
                          size_t ws_bytes, void* stream, bool words32) {
    int rc = check_pipeline_args(c, ell, 1, d, evk, out, ws);
    if (rc != KS_OK) return rc;
    if (words32 && !moduli_fit_u32(c)) return KS_EINVAL;
    if (batch == 0) return KS_OK;
    if (ws_bytes < ks_workspace_bytes(c, KS_OP_KEYSWITCH, ell, batch, 0)) return KS_EWORKSPACE;
    const Level& lv = c->levels[ell - 1];
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint64_t N = c->N, d_ps = (uint64_t)ell * N, out_bs = 2ull * ell * N, word = words32 ? 4 : 8;
    const KsWorkspace one = ks_ws_regions(c, lv, 1);
    const uint32_t chunk = ciphertexts_at_a_time(c, lv, KS_OP_KEYSWITCH, batch, one.coeff + one.lifted + one.acc + one.conv);
    for (uint32_t b0 = 0; b0 < batch; b0 += chunk) {
        const uint32_t bc = std::min(batch - b0, chunk);
        const KsWorkspace w = ks_ws_regions(c, lv, bc);
        uint8_t* coeff = static_cast<uint8_t*>(ws);
        uint8_t* lifted = coeff + w.coeff;
        uint8_t* acc = lifted + w.lifted;
        uint8_t* conv = acc + w.acc;
        const char* dc = static_cast<const char*>(d) + (uint64_t)b0 * d_ps * word;
        const int tile = conversion_tile(c, lv.modup, bc, lv.moddown, 2 * bc);
        mod_up(c, lv, dc, d_ps, coeff, lifted, bc, tile, s, words32);
        key_sums_and_division(c, lv, dc, d_ps, lifted, evk, acc, conv, static_cast<char*>(out) + (uint64_t)b0 * out_bs * word, out_bs, bc, tile, s, (int)word,
                              words32, nullptr, false);
    }
    return finish(words32 ? "ks_keyswitch_u32" : "ks_keyswitch");
}

extern "C" int ks_keyswitch(const ks_ctx* c, const uint64_t* d, uint32_t ell, const uint64_t* evk, uint64_t* out, uint32_t batch,
                            void* ws, size_t ws_bytes, void* stream) {
    return keyswitch_impl(c, d, ell, evk, out, batch, ws, ws_bytes, stream, false);
}

extern "C" int ks_keyswitch_u32(const ks_ctx* c, const uint32_t* d, uint32_t ell, const uint32_t* evk, uint32_t* out, uint32_t batch,
                                void* ws, size_t ws_bytes, void* stream) {
    return keyswitch_impl(c, d, ell, evk, out, batch, ws, ws_bytes, stream, true);
}

// ct, keys and out in 64-bit words, or all in 32-bit words (words32).
static int rotate_hoisted_impl(const ks_ctx* c, const void* ct, uint32_t ell, const uint32_t* galois, const void* const* rot_keys,
                               uint32_t n_rot, void* out, uint32_t batch, void* ws, size_t ws_bytes, void* stream, bool words32) {
    int rc = check_pipeline_args(c, ell, 1, ct, ct, out, ws);
    if (rc != KS_OK) return rc;
    if (!galois || !rot_keys || n_rot == 0) return KS_EINVAL;
    for (uint32_t r = 0; r < n_rot; ++r) {
        if ((galois[r] & 1u) == 0 || galois[r] >= 2u * c->N) return KS_EINVAL;
        if (!rot_keys[r] || !aligned16(rot_keys[r])) return KS_EINVAL;
    }
    if (words32 && !moduli_fit_u32(c)) return KS_EINVAL;
    if (batch == 0) return KS_OK;
    if (ws_bytes < ks_workspace_bytes(c, words32 ? KS_OP_ROTATE_HOISTED_U32 : KS_OP_ROTATE_HOISTED, ell, batch, n_rot))
        return KS_EWORKSPACE;
    const Level& lv = c->levels[ell - 1];
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint64_t N = c->N, ct_bs = 2ull * ell * N, out_bs = (uint64_t)n_rot * 2 * ell * N, word = words32 ? 4 : 8;
    // Rotations of a group: kRotGroup, or where the launches of so many are small, as many as the workspace holds (about eight, see
    // ciphertexts_at_a_time), evenly filled.  Sixteen rotations in groups of four -> eight: N = 2^12, 8 ciphertexts 200 -> 152 us; N = 2^14,
    // 8 ciphertexts 890 -> 816; N = 2^16, one 948 -> 873; but 8 of them 4839 -> 4846 and, 28-bit, 4194 -> 4288; N = 2^15, 8, 28-bit 2083 -> 2140.
    uint32_t group = std::min(n_rot, kRotGroup);
    if (const uint32_t bc = std::min(batch, kChunk); (uint64_t)bc * N < 1u << 18) {
        const KsWorkspace w = ks_ws_regions(c, lv, bc);
        const uint64_t have = ks_workspace_bytes(c, words32 ? KS_OP_ROTATE_HOISTED_U32 : KS_OP_ROTATE_HOISTED, ell, batch, n_rot);
        const uint64_t fixed = gather_words(c, lv, bc, false, words32) * 8 + w.coeff + w.lifted;
        const uint32_t fit = (uint32_t)std::min<uint64_t>(kMacRotations, (have - fixed) / (w.acc + w.conv)), groups = (n_rot + fit - 1) / fit;
        if (groups < (n_rot + kRotGroup - 1) / kRotGroup) group = (n_rot + groups - 1) / groups;
    }
    for (uint32_t b0 = 0; b0 < batch; b0 += kChunk) {
        const uint32_t bc = std::min(batch - b0, kChunk);
        const KsWorkspace w = ks_ws_regions(c, lv, bc);
        // The gathers read c1 and its finished raised digits from a compact bundle; the last kernel's addend c0 is gathered
        // from the ciphertext in its own word size.
        uint64_t* region = static_cast<uint64_t*>(ws);
        uint8_t* coeff = reinterpret_cast<uint8_t*>(region + gather_words(c, lv, bc, false, words32));
        const char* c0 = static_cast<const char*>(ct) + (uint64_t)b0 * ct_bs * word;
        const void* c1 = c0 + (uint64_t)ell * N * word;
        uint8_t* lifted = coeff + w.coeff;
        uint8_t* acc = lifted + w.lifted;
        const int tile = conversion_tile(c, lv.modup, bc, lv.moddown, 2 * group * bc);
        // finished once, shared by every rotation
        const GatherBundle digits = mod_up_for_gather(c, lv, c1, nullptr, ct_bs, coeff, lifted, region, bc, n_rot, tile, s, words32);
        // Rotations go in groups: one gather launch forms the accumulators of the whole group (the raised digits then come
        // from memory once per group), and the inverse transform, the conversion and the last kernel, which adds sigma_g(c0) through
        // each rotation's own permutation, run over the group as one batch.
        uint8_t* conv = acc + (uint64_t)group * w.acc;
        const uint64_t limb = packed_limb_bytes(N), acc_ps = lv.E * limb, conv_ps = ell * limb;
        for (uint32_t r0 = 0; r0 < n_rot; r0 += group) {
            MacRotations rot;
            rot.n = std::min(n_rot - r0, group);
            for (uint32_t r = 0; r < rot.n; ++r) {
                rot.galois[r] = galois[r0 + r];
                rot.key[r] = rot_keys[r0 + r];
                rot.pt[r] = nullptr;
            }
            const bool meet = rotations_meet_division(c, lv, bc, rot.n);
            launch_inner_product(c, lv, digits, rot, acc, s, words32, meet);
            const uint32_t polys = 2 * rot.n * bc;
            launch_inv_rows_packed(c, lv.special_map, acc, acc_ps, 1, acc, acc_ps, polys, s);
            launch_inv_cols_packed(c, lv.special_map, acc, acc_ps, polys, c->d_moddown_scale, s);
            launch_bconv_ntt_cols(c, lv.moddown, c->K + lv.ell, acc, acc_ps, conv, conv_ps, polys, tile, s);
            char* to = static_cast<char*>(out) + ((uint64_t)b0 * out_bs + (uint64_t)r0 * 2 * ell * N) * word;
            if (meet) launch_rotate_finish(c, lv, digits, rot, conv, to, out_bs, c0, s, words32);
            else launch_rows_moddown_finish(c, lv, acc, conv, to, out_bs, c0, ct_bs, &rot, 2ull * ell * N, bc, s, nullptr, words32);
        }
    }
    return finish(words32 ? "ks_rotate_hoisted_u32" : "ks_rotate_hoisted");
}

extern "C" int ks_rotate_hoisted(const ks_ctx* c, const uint64_t* ct, uint32_t ell, const uint32_t* galois,
                                 const uint64_t* const* rot_keys, uint32_t n_rot, uint64_t* out, uint32_t batch, void* ws,
                                 size_t ws_bytes, void* stream) {
    return rotate_hoisted_impl(c, ct, ell, galois, reinterpret_cast<const void* const*>(rot_keys), n_rot, out, batch, ws, ws_bytes,
                               stream, false);
}

extern "C" int ks_rotate_hoisted_u32(const ks_ctx* c, const uint32_t* ct, uint32_t ell, const uint32_t* galois,
                                     const uint32_t* const* rot_keys, uint32_t n_rot, uint32_t* out, uint32_t batch, void* ws,
                                     size_t ws_bytes, void* stream) {
    return rotate_hoisted_impl(c, ct, ell, galois, reinterpret_cast<const void* const*>(rot_keys), n_rot, out, batch, ws, ws_bytes,
                               stream, true);
}

// Galois elements, keys and plaintexts of a rotate-multiply-accumulate: g = 1 needs no key, a null plaintext is 1.
static int check_mac_rotations(const ks_ctx* c, const uint32_t* galois, const void* const* keys, const void* const* pts,
                               uint32_t n) {
    if (!galois || !keys || n == 0) return KS_EINVAL;
    for (uint32_t r = 0; r < n; ++r) {
        if ((galois[r] & 1u) == 0 || galois[r] >= 2u * c->N) return KS_EINVAL;
        if (galois[r] != 1 && (!keys[r] || !aligned16(keys[r]))) return KS_EINVAL;
        if (pts && pts[r] && !aligned16(pts[r])) return KS_EINVAL;
    }
    return KS_OK;
}

// u (+)= sum_r pt_r * rot_{g_r}(ct) for all n rotations, in launches of kMacRotations
static void rotate_mac_all(const ks_ctx* c, const Level& lv, const GatherBundle& src,
                           const uint32_t* galois, const void* const* keys, const void* const* pts, uint32_t n, uint8_t* u,
                           bool accumulate, hipStream_t s, bool key_words32 = false) {
    for (uint32_t r0 = 0; r0 < n; r0 += kMacRotations) {
        MacRotations rot;
        rot.n = std::min<uint32_t>(n - r0, kMacRotations);
        for (uint32_t r = 0; r < rot.n; ++r) {
            rot.galois[r] = galois[r0 + r];
            rot.key[r] = keys[r0 + r];
            rot.pt[r] = pts ? pts[r0 + r] : nullptr;
        }
        launch_rotate_mac(c, lv, src, rot, u, accumulate || r0 != 0, s, key_words32);
    }
}

// u_i = sum_r pt_{i, r} * rot_{g_r}(ct) for n rows of diagonals (ptv [n][n_rot]), u_i u_stride bytes apart
static void rotate_mac_rows_all(const ks_ctx* c, const Level& lv, const GatherBundle& src, const uint32_t* galois, const void* const* keys,
                                const void* const* ptv, uint32_t n_rot, uint32_t n, uint8_t* u, uint64_t u_stride, hipStream_t s, bool key_words32) {
    for (uint32_t r0 = 0; r0 < n_rot; r0 += kMacRotations) {
        MacRotations rot{};
        MacRows rows{};
        rot.n = std::min<uint32_t>(n_rot - r0, kMacRotations);
        rows.n = n;
        for (uint32_t r = 0; r < rot.n; ++r) {
            rot.galois[r] = galois[r0 + r];
            rot.key[r] = keys[r0 + r];
            for (uint32_t i = 0; i < n; ++i) rows.pt[i][r] = ptv[(size_t)i * n_rot + r0 + r];
        }
        launch_rotate_mac_rows(c, lv, src, rot, rows, u, u_stride, r0 != 0, s, key_words32);
    }
}

static int rotate_mac_impl(const ks_ctx* c, const void* ct, uint32_t ell, const uint32_t* galois, const void* const* rot_keys,
                           const void* const* pts, uint32_t n_rot, void* out, uint32_t batch, void* ws, size_t ws_bytes, void* stream,
                           bool words32) {
    int rc = check_pipeline_args(c, ell, 1, ct, ct, out, ws);
    if (rc != KS_OK) return rc;
    if (!pts || (rc = check_mac_rotations(c, galois, rot_keys, pts, n_rot)) != KS_OK) return KS_EINVAL;
    if (words32 && !moduli_fit_u32(c)) return KS_EINVAL;
    if (batch == 0) return KS_OK;
    if (ws_bytes < ks_workspace_bytes(c, words32 ? KS_OP_ROTATE_HOISTED_U32 : KS_OP_ROTATE_HOISTED, ell, batch, n_rot))
        return KS_EWORKSPACE;
    const Level& lv = c->levels[ell - 1];
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint64_t N = c->N, ct_bs = 2ull * ell * N, word = words32 ? 4 : 8;
    for (uint32_t b0 = 0; b0 < batch; b0 += kChunk) {
        const uint32_t bc = std::min(batch - b0, kChunk);
        const KsWorkspace w = ks_ws_regions(c, lv, bc);
        // the gathers read c1 and its finished raised digits, and c0 for many rotations, from a compact bundle
        const char* c0 = static_cast<const char*>(ct) + (uint64_t)b0 * ct_bs * word;
        uint64_t* region = static_cast<uint64_t*>(ws);
        uint8_t* coeff = reinterpret_cast<uint8_t*>(region + gather_words(c, lv, bc, n_rot >= kC0InBundle, words32));
        uint8_t* lifted = coeff + w.coeff;
        uint8_t* acc = lifted + w.lifted;
        uint8_t* conv = acc + w.acc;
        const int tile = conversion_tile(c, lv.modup, bc, lv.moddown, 2 * bc);
        // finished once, shared by every rotation
        const GatherBundle digits = mod_up_for_gather(c, lv, c0 + (uint64_t)ell * N * word, c0, ct_bs, coeff, lifted, region, bc, n_rot, tile, s, words32);
        rotate_mac_all(c, lv, digits, galois, rot_keys, pts, n_rot, acc, false, s, words32);
        mod_down(c, lv, acc, conv, static_cast<char*>(out) + (uint64_t)b0 * ct_bs * word, ct_bs, bc, tile, s, words32);
    }
    return finish(words32 ? "ks_rotate_mac_hoisted_u32" : "ks_rotate_mac_hoisted");
}

extern "C" int ks_rotate_mac_hoisted(const ks_ctx* c, const uint64_t* ct, uint32_t ell, const uint32_t* galois,
                                     const uint64_t* const* rot_keys, const uint64_t* const* pts, uint32_t n_rot, uint64_t* out,
                                     uint32_t batch, void* ws, size_t ws_bytes, void* stream) {
    return rotate_mac_impl(c, ct, ell, galois, reinterpret_cast<const void* const*>(rot_keys),
                           reinterpret_cast<const void* const*>(pts), n_rot, out, batch, ws, ws_bytes, stream, false);
}

extern "C" int ks_rotate_mac_hoisted_u32(const ks_ctx* c, const uint32_t* ct, uint32_t ell, const uint32_t* galois,
                                         const uint32_t* const* rot_keys, const uint32_t* const* pts, uint32_t n_rot, uint32_t* out,
                                         uint32_t batch, void* ws, size_t ws_bytes, void* stream) {
    return rotate_mac_impl(c, ct, ell, galois, reinterpret_cast<const void* const*>(rot_keys),
                           reinterpret_cast<const void* const*>(pts), n_rot, out, batch, ws, ws_bytes, stream, true);
}

// ct, keys, plaintexts and out in 64-bit words, or all in 32-bit words (words32).
static int bsgs_impl(const ks_ctx* c, const void* ct, uint32_t ell, const uint32_t* baby_galois, const void* const* bkeys, uint32_t n1,
                     const uint32_t* giant_galois, const void* const* gkeys, uint32_t n2, const void* const* ptv, void* out,
                     uint32_t batch, void* ws, size_t ws_bytes, void* stream, bool words32) {
    int rc = check_pipeline_args(c, ell, 1, ct, ct, out, ws);
    if (rc != KS_OK) return rc;
    if (!ptv || check_mac_rotations(c, giant_galois, gkeys, nullptr, n2) != KS_OK) return KS_EINVAL;
    for (uint32_t g = 0; g < n2; ++g)
        if (check_mac_rotations(c, baby_galois, bkeys, ptv + (size_t)g * n1, n1) != KS_OK) return KS_EINVAL;
    if (words32 && !moduli_fit_u32(c)) return KS_EINVAL;
    if (batch == 0) return KS_OK;
    if (ws_bytes < ks_workspace_bytes(c, words32 ? KS_OP_BSGS_U32 : KS_OP_BSGS, ell, batch, 0)) return KS_EWORKSPACE;
    const Level& lv = c->levels[ell - 1];
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint64_t N = c->N, ct_bs = 2ull * ell * N, word = words32 ? 4 : 8;
    for (uint32_t b0 = 0; b0 < batch; b0 += kChunk) {
        const uint32_t bc = std::min(batch - b0, kChunk);
        const KsWorkspace w = ks_ws_regions(c, lv, bc);
        // The gathers of the inner level read the input ciphertext and its finished raised digits from a compact bundle; the
        // inner results are 64-bit words either way, so the outer level's bundle is the packed one.
        const char* c0 = static_cast<const char*>(ct) + (uint64_t)b0 * ct_bs * word;
        uint64_t* region = static_cast<uint64_t*>(ws);   // sources of the inner level, shared by every baby step of every giant step
        uint64_t* region_v = region + gather_words(c, lv, bc, true, words32);   // sources of the outer level: the current inner result
        uint8_t* coeff = reinterpret_cast<uint8_t*>(region_v + gather_words(c, lv, bc, false, false));
        uint8_t* lifted = coeff + w.coeff;          // scratch of a ModUp
        uint8_t* conv = lifted + w.lifted;
        uint8_t* acc_outer = conv + w.conv;         // outer sum over the giant steps
        uint64_t* v = reinterpret_cast<uint64_t*>(acc_outer + w.acc);   // [bc][2][ell][N] inner result of the current giant step (64-bit words)
        uint8_t* acc = reinterpret_cast<uint8_t*>(v + (uint64_t)bc * 2 * ell * N);   // inner sums of the giant steps at hand
        const int tile = conversion_tile(c, lv.modup, bc, lv.moddown, 2 * bc);
        const GatherBundle digits = mod_up_for_gather(c, lv, c0 + (uint64_t)ell * N * word, c0, ct_bs, coeff, lifted, region, bc, n1 * n2, tile, s, words32);
        // Inner sums of four or two giant steps at a time where the workspace holds them (a caller brings what ks_workspace_bytes asks for, 8
        // bytes a residue: four of three digits, three of two digits with a short second one and of one digit) and the bundle has c0.  Groups of
        // more than four are two halves there, which have to pay with shared keys for what they load twice: four rows, more than one digit (and
        // one digit has little to share: up to two ciphertexts).  Eight baby and four giant steps, N = 2^16, us by rows at a time, 1 / 2 / 4:
        // three digits, one ciphertext 1220 / 980 / 822, four 2423 / 2180 / 1908, five 2905 / 3025 / 2583, eight 4143 / 4347 / 3638; two digits,
        // four 1884 / 1737 / 1563, eight 3253 / 3438 / 2967; one digit, one 595 / 537, four 1161 / 1152, eight 2023 / 2217; 28 bits, three
        // digits, one 894 / 772 / 672, eight 3627 / 3443 / 3215.  Few baby steps gain less but gain, one row -> rows at a time: three digits, 24
        // limbs, two baby steps, four ciphertexts 2116 -> 2007, eight 6279 -> 6017, four baby steps, three 2340 -> 2100, eight 3481 -> 3230;
        // two digits, two baby steps, one (8 limbs) 329 -> 312, four (11 limbs) 1159 -> 1151; N = 2^15, 9 limbs, one 284 -> 267, four 639 -> 625.
        const uint64_t have = ks_workspace_bytes(c, words32 ? KS_OP_BSGS_U32 : KS_OP_BSGS, ell, bc, 0), used = acc - static_cast<uint8_t*>(ws);
        const uint64_t fit = digits.c0 ? 1 : (have - used) / w.acc;
        const bool small = bc <= (lv.ndig > 1 ? 4 : 2), rows4 = fit >= kMacRows && (small || lv.ndig > 1), rows2 = fit >= 2 && small;
        for (uint32_t g0 = 0, n; g0 < n2; g0 += n) {
            n = rows4 && n2 - g0 >= kMacRows ? kMacRows : rows2 && n2 - g0 >= 2 ? 2 : 1;
            const void* const* pts = ptv + (size_t)g0 * n1;
            if (n == 1) rotate_mac_all(c, lv, digits, baby_galois, bkeys, pts, n1, acc, false, s, words32);
            else rotate_mac_rows_all(c, lv, digits, baby_galois, bkeys, pts, n1, n, acc, w.acc, s, words32);
            for (uint32_t i = 0; i < n; ++i) {
                const uint32_t g = g0 + i;
                mod_down(c, lv, acc + i * w.acc, conv, v, ct_bs, bc, tile, s);
                const GatherBundle digits_v = mod_up_for_gather(c, lv, v + (uint64_t)ell * N, v, ct_bs, coeff, lifted, region_v, bc, 1, tile, s, false,
                                                                giant_galois[g] != 1);
                rotate_mac_all(c, lv, digits_v, giant_galois + g, gkeys + g, nullptr, 1, acc_outer, g != 0, s, words32);
            }
        }
        mod_down(c, lv, acc_outer, conv, static_cast<char*>(out) + (uint64_t)b0 * ct_bs * word, ct_bs, bc, tile, s,
                 words32);
    }
    return finish(words32 ? "ks_bsgs_linear_transform_u32" : "ks_bsgs_linear_transform");
}

extern "C" int ks_bsgs_linear_transform(const ks_ctx* c, const uint64_t* ct, uint32_t ell, const uint32_t* baby_galois,
                                        const uint64_t* const* baby_keys, uint32_t n1, const uint32_t* giant_galois,
                                        const uint64_t* const* giant_keys, uint32_t n2, const uint64_t* const* pts, uint64_t* out,
                                        uint32_t batch, void* ws, size_t ws_bytes, void* stream) {
    return bsgs_impl(c, ct, ell, baby_galois, reinterpret_cast<const void* const*>(baby_keys), n1, giant_galois,
                     reinterpret_cast<const void* const*>(giant_keys), n2, reinterpret_cast<const void* const*>(pts), out, batch, ws,
                     ws_bytes, stream, false);
}

extern "C" int ks_bsgs_linear_transform_u32(const ks_ctx* c, const uint32_t* ct, uint32_t ell, const uint32_t* baby_galois,
                                            const uint32_t* const* baby_keys, uint32_t n1, const uint32_t* giant_galois,
                                            const uint32_t* const* giant_keys, uint32_t n2, const uint32_t* const* pts, uint32_t* out,
                                            uint32_t batch, void* ws, size_t ws_bytes, void* stream) {
    return bsgs_impl(c, ct, ell, baby_galois, reinterpret_cast<const void* const*>(baby_keys), n1, giant_galois,
                     reinterpret_cast<const void* const*>(giant_keys), n2, reinterpret_cast<const void* const*>(pts), out, batch, ws,
                     ws_bytes, stream, true);
}

// cta, ctb, rlk and out in 64-bit words, or all four in 32-bit words (words32).
static int hmult_impl(const ks_ctx* c, const void* cta, const void* ctb, uint32_t ell, const void* rlk, void* out, uint32_t batch,
                      void* ws, size_t ws_bytes, void* stream, bool merged, bool words32) {
    int rc = check_pipeline_args(c, ell, 2, cta, ctb, out, ws);
    if (rc != KS_OK) return rc;
    if (!rlk || !aligned16(rlk)) return KS_EINVAL;
    if (words32 && !moduli_fit_u32(c)) return KS_EINVAL;
    if (batch == 0) return KS_OK;
    if (ws_bytes < ks_workspace_bytes(c, KS_OP_HMULT_RELIN_RESCALE, ell, batch, 0)) return KS_EWORKSPACE;
    const Level& lv = c->levels[ell - 1];
    if (merged && !lv.merged.d_plans) return KS_EINVAL;  // K + 1 sources exceed what one conversion takes
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint64_t N = c->N, ct_bs = 2ull * ell * N, out_bs = 2ull * (ell - 1) * N, word = words32 ? 4 : 8;
    const KsWorkspace one = ks_ws_regions(c, lv, 1);
    // (d0, d1) as large as conv, d2 as coeff
    const uint32_t chunk = ciphertexts_at_a_time(c, lv, KS_OP_HMULT_RELIN_RESCALE, batch, 2 * one.coeff + one.lifted + one.acc + 2 * one.conv);
    for (uint32_t b0 = 0; b0 < batch; b0 += chunk) {
        const uint32_t bc = std::min(batch - b0, chunk);
        const KsWorkspace w = ks_ws_regions(c, lv, bc);
        uint8_t* coeff = static_cast<uint8_t*>(ws);
        uint8_t* lifted = coeff + w.coeff;
        uint8_t* acc = lifted + w.lifted;
        uint8_t* conv = acc + w.acc;
        uint8_t* dq = conv + w.conv;                                    // (d0, d1): [bc][2][ell] packed
        uint8_t* d2 = dq + w.conv;                                      // [bc][ell] packed, the polynomial that is key-switched
        char* oc = static_cast<char*>(out) + (uint64_t)b0 * out_bs * word;
        launch_tensor_inv_rows(c, static_cast<const char*>(cta) + (uint64_t)b0 * ct_bs * word,
                               static_cast<const char*>(ctb) + (uint64_t)b0 * ct_bs * word, ell, dq, d2, coeff, bc, s, words32);
        const int tile = conversion_tile(c, lv.modup, bc, merged ? lv.merged : lv.rescale, 2 * bc);
        mod_up_from_rows(c, lv, coeff, lifted, bc, tile, s);
        key_sums_and_division(c, lv, d2, w.coeff / bc, lifted, rlk, acc, conv, oc, out_bs, bc, tile, s, 1, words32, dq, merged);
    }
    if (merged) return finish(words32 ? "hmult_relin_rescale_merged_u32" : "hmult_relin_rescale_merged");
    return finish(words32 ? "hmult_relin_rescale_u32" : "hmult_relin_rescale");
}

extern "C" int hmult_relin_rescale_merged(const ks_ctx* c, const uint64_t* cta, const uint64_t* ctb, uint32_t ell, const uint64_t* rlk,
                                          uint64_t* out, uint32_t batch, void* ws, size_t ws_bytes, void* stream) {
    return hmult_impl(c, cta, ctb, ell, rlk, out, batch, ws, ws_bytes, stream, true, false);
}

extern "C" int hmult_relin_rescale(const ks_ctx* c, const uint64_t* cta, const uint64_t* ctb, uint32_t ell, const uint64_t* rlk,
                                   uint64_t* out, uint32_t batch, void* ws, size_t ws_bytes, void* stream) {
    return hmult_impl(c, cta, ctb, ell, rlk, out, batch, ws, ws_bytes, stream, false, false);
}

extern "C" int hmult_relin_rescale_merged_u32(const ks_ctx* c, const uint32_t* cta, const uint32_t* ctb, uint32_t ell,
                                              const uint32_t* rlk, uint32_t* out, uint32_t batch, void* ws, size_t ws_bytes,
                                              void* stream) {
    return hmult_impl(c, cta, ctb, ell, rlk, out, batch, ws, ws_bytes, stream, true, true);
}

extern "C" int hmult_relin_rescale_u32(const ks_ctx* c, const uint32_t* cta, const uint32_t* ctb, uint32_t ell, const uint32_t* rlk,
                                       uint32_t* out, uint32_t batch, void* ws, size_t ws_bytes, void* stream) {
    return hmult_impl(c, cta, ctb, ell, rlk, out, batch, ws, ws_bytes, stream, false, true);
}
