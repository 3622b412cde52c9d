// sa_block_forward: one pass of the reparameterised block (Eq. 2 restricted to the
// attention MatMuls and the MLP): hash Q and K, additive or Hamming attention, then the
// Shift MLP or the two-expert MoE.  A composition of the library's own steps; the expert row counts
// stay on the device (no host round trip).
#include "common.h"
#include "gemm_common.h"

namespace {

struct Layout {
    size_t qc, kc, kv, attn_ws, xq, xh, perm, expert_of, counts, gate, disp_ws, shift_ws, mult_ws, needed, few, total;
    size_t attn_ws_bytes, disp_ws_bytes, shift_ws_bytes, mult_ws_bytes;
};

size_t up(size_t x) { return (x + 255) / 256 * 256; }

int plan(const sa_block_desc *d, Layout *L) {
    SA_REQUIRE(d != nullptr, SA_ERR_INVALID, "block: descriptor is NULL");
    SA_REQUIRE(d->B > 0 && d->N > 0 && d->H > 0 && d->d > 0 && d->nbits > 0 && d->dv > 0, SA_ERR_INVALID,
               "block: sizes must be positive");
    SA_REQUIRE(d->nbits % 64 == 0, SA_ERR_SHAPE, "block: nbits must be a multiple of 64");
    SA_REQUIRE(d->attention == 0 || d->attention == 1, SA_ERR_INVALID, "block: attention must be 0 or 1");
    SA_REQUIRE(d->hid >= 0, SA_ERR_INVALID, "block: hid < 0");
    const size_t T = (size_t)d->B * d->N, E = (size_t)d->H * d->dv;
    SA_REQUIRE(T < (1ull << 31), SA_ERR_SHAPE, "block: too many tokens");
    size_t off = 0;
    const size_t code_bytes = up((size_t)d->B * d->H * d->N * (d->nbits / 64) * 8);
    L->qc = off; off += code_bytes;
    L->kc = off; off += code_bytes;
    L->kv = off;
    L->attn_ws_bytes = 0;
    if (d->attention == 0) {
        off += up((size_t)d->B * d->H * d->nbits * d->dv * 4);
        L->attn_ws_bytes = sa_additive_attention_workspace_bytes(d->B, d->H, d->N, d->nbits, d->dv);
    }
    L->attn_ws = off; off += up(L->attn_ws_bytes);
    L->xq = L->xh = off;
    L->disp_ws_bytes = L->shift_ws_bytes = L->mult_ws_bytes = 0;
    L->perm = L->expert_of = L->counts = L->gate = L->disp_ws = L->shift_ws = L->mult_ws = off;
    if (d->hid > 0) {
        off += up(T * E);
        L->shift_ws_bytes = sa_shift_mlp_workspace_bytes((long)T, (int)E, d->hid);
        L->shift_ws = off; off += up(L->shift_ws_bytes);
        if (d->moe) {
            L->xh = off; off += up(T * E * 2);          // fp16 copy of the attention output for the Mult expert
            L->perm = off; off += up(T * 4);
            L->expert_of = off; off += up(T * 4);
            L->counts = off; off += 256;
            L->gate = off; off += up(T * 4);
            L->disp_ws_bytes = sa_moe_dispatch_workspace_bytes((long)T, 2);
            L->disp_ws = off; off += up(L->disp_ws_bytes);
            L->mult_ws_bytes = sa_mult_mlp_workspace_bytes((long)T, (int)E, d->hid);
            L->mult_ws = off; off += up(L->mult_ws_bytes);
        }
    }
    L->needed = L->few = off;
    if (d->hid > 0) off += up(sa::plan_few_rows((long)T, (int)E, d->hid, d->moe != 0, false).bytes);
    L->total = off;
    return SA_OK;
}

}  // namespace

extern "C" size_t sa_block_workspace_bytes(const sa_block_desc *desc) {
    Layout L;
    if (plan(desc, &L) != SA_OK) return 0;
    return L.total;
}

namespace {

// What the MLP asks of its operands.
template <class Desc>
int check_mlp(const Desc &d, int E, long T) {
    SA_REQUIRE(d.shift_variant >= 0 && d.shift_variant <= 3, SA_ERR_INVALID, "MLP: unknown shift variant %d", d.shift_variant);
    SA_REQUIRE(E % 64 == 0 && d.hid % 64 == 0, SA_ERR_SHAPE, "MLP: E (%d) and hid (%d) must be multiples of 64", E, d.hid);
    SA_REQUIRE(E <= 131072 && d.hid <= 131072, SA_ERR_SHAPE, "MLP: width too large");
    SA_REQUIRE(sa::aligned16(d.w1) && sa::aligned16(d.w2) && sa::aligned16(d.lut) && sa::aligned16(d.y) &&
                   (!d.moe || (sa::aligned16(d.mw1) && sa::aligned16(d.mw2))),
               SA_ERR_ALIGN, "MLP: pointers must be 16-byte aligned");
    SA_REQUIRE(sa::shift_rows_fit(T, d.shift_variant), SA_ERR_SHAPE, "MLP: too many rows for the VALU variant in one call");
    return SA_OK;
}

// The Shift weights of an MLP as its layers take them: packed ones that the matrix cores need decoded become a job for a
// launch before the MLP, and the planes that job fills take their place (the prepared variant).
struct ShiftWeights {
    const uint8_t *w1, *w2;
    int variant;
    template <class Desc>
    ShiftWeights(const Desc &d, int E, long T, void *shift_ws, sa::DecodeWork *work) : w1(d.w1), w2(d.w2), variant(d.shift_variant) {
        if (variant != SA_VARIANT_MFMA && variant != SA_VARIANT_AUTO) return;
        sa::shift_mlp_decode(work, d.w1, d.w2, E, d.hid, T, shift_ws, &w1, &w2);
        variant = SA_VARIANT_MFMA_PREPARED;
    }
};

// Whether the MLP of this block, or the MLP half of this layer, is one launch: with few rows on the matrix cores, where the caller's
// workspace has room for it (the size that is asked for does; a smaller one is taken as long as the other launches' fits).
template <class Desc>
sa::FewRowsPlan few_rows(const Desc &d, int E, long T, bool layer, size_t workspace_bytes) {
    if (d.hid <= 0 || d.shift_variant == SA_VARIANT_VALU || d.workspace_bytes < workspace_bytes) return {};
    return sa::plan_few_rows(T, E, d.hid, d.moe != 0, layer);
}

// Hash of Q and K, carrying `side` where it is one launch, and in any case what is to be cleared (a launch for that alone took
// more than few rows and the sign hash gain by it: Shift block of 784 x 64, 512 hidden 19.6 -> 22.6 us, without that launch 17.8 -> 16.4; of 784 x
// 128 21.1 -> 21.6).
int hash_and_side(const float *q, const float *k, int B, int N, int H, int d, const float *proj, int nbits, uint64_t *qc,
                  uint64_t *kc, const sa::SideWork &side, void *stream) {
    if (side.any() && sa::binarize_pair_one_launch(q, k, proj, qc, kc, (long)B * N * H, d, nbits))
        return sa::launch_binarize_mfma(q, k, proj, qc, kc, (long)B * N * H, N, H, d, nbits, sa::as_stream(stream), side);
    int rc = SA_OK;
    const sa::RouteWork &r = side.route;
    if (r.T > 0) rc = sa::moe_dispatch_launch(r.logits, r.T, r.E, r.perm, r.expert_of, r.counts, r.gate, nullptr, sa::as_stream(stream));
    if (rc == SA_OK && side.decode.chunks[0] > 0) rc = sa::launch_decode_work(side.decode, sa::as_stream(stream));
    if (rc != SA_OK) return rc;
    if (!proj) return sa::launch_sign_pair(q, k, (long)B * N * H, N, H, d, qc, kc, side.zero, sa::as_stream(stream));
    if (side.zero.n > 0) rc = sa::launch_zero(side.zero.words, 4 * (size_t)side.zero.n, sa::as_stream(stream));
    if (rc != SA_OK) return rc;
    return sa_binarize_pair(q, k, B, N, H, d, proj, nbits, qc, kc, stream);
}

// The two experts of a block or layer, on the rows the routing gave them.  On the matrix cores both run in the same
// launches, layer by layer; the Shift expert's vector-ALU variant has launches of its own.
template <class Desc>
int experts(const Desc &d, const ShiftWeights &w, const int8_t *xq, const void *xh, int E, long T, const int32_t *perm,
            const int32_t *counts, const float *gate, int flags, void *mult_ws, size_t mult_ws_bytes, void *shift_ws,
            size_t shift_ws_bytes, void *stream) {
    const sa_rows mult_rows{perm, counts, 0, T}, shift_rows{perm, counts, 1, T};
    if (w.variant == SA_VARIANT_MFMA_PREPARED) {
        sa::ExpertPair p{xq, xh, {}, {}, d.y, gate, d.out_scale};
        int rc = sa::validate_rows(&shift_rows, &p.shift_rows);
        if (rc == SA_OK) rc = sa::validate_rows(&mult_rows, &p.mult_rows);
        if (rc != SA_OK) return rc;
        return sa::expert_pair_mlp(p, E, d.hid, reinterpret_cast<const int8_t *>(w.w1), reinterpret_cast<const int8_t *>(w.w2), d.mw1,
                                   d.mw2, d.requant_scale, d.lut, flags != 0, static_cast<int8_t *>(shift_ws), mult_ws,
                                   sa::as_stream(stream));
    }
    int rc = sa_mult_mlp_f16_half(xh, &mult_rows, E, d.hid, d.mw1, d.mw2, nullptr, d.y, gate, 3 | flags, mult_ws, mult_ws_bytes,
                                  stream);
    if (rc != SA_OK) return rc;
    return sa_shift_mlp(xq, &shift_rows, E, d.hid, w.w1, w.w2, d.requant_scale, d.lut, nullptr, d.y, gate, d.out_scale, w.variant,
                        3 | flags, shift_ws, shift_ws_bytes, stream);
}

}  // namespace

extern "C" int sa_block_forward(const sa_block_desc *d, void *stream) {
    sa::clear_error();
    Layout L;
    int rc = plan(d, &L);
    if (rc != SA_OK) return rc;
    SA_REQUIRE(d->q && d->k && d->v && d->o, SA_ERR_INVALID, "block: q, k, v and o are required");
    SA_REQUIRE(d->workspace != nullptr && d->workspace_bytes >= L.needed, SA_ERR_WORKSPACE,
               "block: workspace of %zu bytes asked for, %zu needed, %zu given", L.total, L.needed, d->workspace_bytes);
    SA_REQUIRE(sa::aligned16(d->workspace), SA_ERR_ALIGN, "block: workspace must be 16-byte aligned");
    if (d->hid > 0) {
        SA_REQUIRE(d->w1 && d->w2 && d->lut && d->y, SA_ERR_INVALID, "block: w1, w2, lut and y are required");
        if (d->moe) SA_REQUIRE(d->logits && d->mw1 && d->mw2, SA_ERR_INVALID, "block: logits, mw1, mw2 are required");
    }
    uint8_t *ws = static_cast<uint8_t *>(d->workspace);
    uint64_t *qc = reinterpret_cast<uint64_t *>(ws + L.qc), *kc = reinterpret_cast<uint64_t *>(ws + L.kc);
    const long T = (long)d->B * d->N;
    const int E = d->H * d->dv;

    const bool moe = d->hid > 0 && d->moe;
    int32_t *perm = reinterpret_cast<int32_t *>(ws + L.perm);
    int32_t *expert_of = reinterpret_cast<int32_t *>(ws + L.expert_of);
    int32_t *counts = reinterpret_cast<int32_t *>(ws + L.counts);
    float *gate = reinterpret_cast<float *>(ws + L.gate);
    int8_t *xq = reinterpret_cast<int8_t *>(ws + L.xq);
    void *xh = moe ? static_cast<void *>(ws + L.xh) : nullptr;
    const bool mlp = d->hid > 0;
    float *kv = reinterpret_cast<float *>(ws + L.kv);

    // Every step's arguments are checked before the first launch.
    rc = sa::check_binarize_pair(d->q, d->k, d->B, d->N, d->H, d->d, d->proj, d->nbits, qc, kc);
    if (rc == SA_OK)
        rc = d->attention == 0 ? sa::check_additive_attention(qc, kc, d->v, d->o, d->B, d->H, d->N, d->N, d->nbits, d->dv, kv, 3,
                                                              ws + L.attn_ws, L.attn_ws_bytes)
                               : sa::check_hamming_attention(qc, kc, d->v, d->o, d->B, d->H, d->N, d->N, d->nbits, d->dv, d->attn_scale,
                                                             nullptr, mlp ? xq : nullptr, xh, SA_VARIANT_AUTO);
    if (rc == SA_OK && mlp) rc = check_mlp(*d, E, T);
    if (rc == SA_OK && moe)
        rc = sa::check_moe_dispatch(d->logits, T, 2, perm, expert_of, counts, gate, ws + L.disp_ws, L.disp_ws_bytes);
    if (rc != SA_OK) return rc;

    // Everything runs on the caller's stream, one kernel after the other.
    // The routing and the decode of packed Shift weights wait for nothing: they ride in the hash's launch.
    sa::SideWork side;
    const sa::FewRowsPlan plan = few_rows(*d, E, T, false, L.total);
    const bool few = plan.bytes > 0;
    if (few) {
        side.zero = {reinterpret_cast<uint32_t *>(ws + L.few), (int)(plan.ticket_bytes / 4)};
    } else if (moe && T <= sa::kSideRouteTokens) {
        side.route = {d->logits, T, 2, expert_of, gate, counts, perm};
    } else if (moe) {
        rc = sa_moe_dispatch(d->logits, T, 2, perm, expert_of, counts, gate, ws + L.disp_ws, L.disp_ws_bytes, stream);
        if (rc != SA_OK) return rc;
    }
    sa::DecodeWork none;
    const ShiftWeights weights(*d, E, T, ws + L.shift_ws, mlp ? &side.decode : &none);
    rc = hash_and_side(d->q, d->k, d->B, d->N, d->H, d->d, d->proj, d->nbits, qc, kc, side, stream);
    if (rc != SA_OK) return rc;
    // The attention output leaves in three forms: fp32 (the block's output o), the int8 codes the
    // Shift layers read, and (with a Mult expert) the fp16 rounding its first layer reads.  The
    // kernel that computes it writes all three from its accumulators.
    if (d->attention == 0) {
        rc = sa::additive_attention_fused(qc, kc, d->v, d->o, true, d->B, d->H, d->N, d->nbits, d->dv, d->attn_scale, kv,
                                          mlp ? xq : nullptr, static_cast<_Float16 *>(xh), d->act_inv_scale, ws + L.attn_ws,
                                          L.attn_ws_bytes, stream);
    } else {
        rc = sa_hamming_attention_fused(qc, kc, d->v, d->o, d->B, d->H, d->N, d->N, d->nbits, d->dv, d->attn_scale,
                                         nullptr, mlp ? xq : nullptr, xh, d->act_inv_scale, SA_VARIANT_AUTO, stream);
    }
    if (rc != SA_OK || !mlp) return rc;

    if (few)
        return sa::launch_few_rows({xq, xh, nullptr, nullptr, nullptr, moe ? d->logits : nullptr, T, E, d->hid, reinterpret_cast<const int8_t *>(weights.w1),
                                    reinterpret_cast<const int8_t *>(weights.w2), d->lut, moe ? d->mw1 : nullptr, moe ? d->mw2 : nullptr,
                                    d->requant_scale, d->out_scale, d->y, ws + L.few}, plan, sa::as_stream(stream));
    if (!moe) {
        const sa_rows all{nullptr, nullptr, 0, T};
        return sa_shift_mlp(xq, &all, E, d->hid, weights.w1, weights.w2, d->requant_scale, d->lut, nullptr, d->y, nullptr,
                            d->out_scale, weights.variant, 3, ws + L.shift_ws, L.shift_ws_bytes, stream);
    }
    return experts(*d, weights, xq, xh, E, T, perm, counts, gate, 0, ws + L.mult_ws, L.mult_ws_bytes, ws + L.shift_ws, L.shift_ws_bytes,
                   stream);
}

// ---------------------------------------------------------------------------------------
// sa_layer_forward: the complete block of Eq. 2.  LayerNorm -> int8 -> fused Q/K/V shift
// Linear -> hash -> attention -> int8 -> output shift Linear + residual -> LayerNorm (int8,
// fp16 and router logits in one pass) -> dispatch -> experts adding into the residual rows.
namespace {

struct LayerLayout {
    size_t codes8, q, k, v, qc, kc, kv, attn_ws, xh, logits, perm, expert_of, counts, gate, disp_ws, shift_ws,
        mult_ws, lin_ws, needed, few, few_wo, total;
    size_t attn_ws_bytes, disp_ws_bytes, shift_ws_bytes, mult_ws_bytes, lin_ws_bytes;
};

int plan_layer(const sa_layer_desc *d, LayerLayout *L) {
    SA_REQUIRE(d != nullptr, SA_ERR_INVALID, "layer: descriptor is NULL");
    SA_REQUIRE(d->B > 0 && d->N > 0 && d->H > 0 && d->nbits > 0 && d->E > 0 && d->hid > 0, SA_ERR_INVALID,
               "layer: sizes must be positive");
    SA_REQUIRE(d->E % d->H == 0, SA_ERR_SHAPE, "layer: E (%d) is not a multiple of H (%d)", d->E, d->H);
    SA_REQUIRE(d->E % 64 == 0 && d->hid % 64 == 0, SA_ERR_SHAPE, "layer: E and hid must be multiples of 64");
    SA_REQUIRE(d->nbits % 64 == 0, SA_ERR_SHAPE, "layer: nbits must be a multiple of 64");
    SA_REQUIRE(d->attention == 0 || d->attention == 1, SA_ERR_INVALID, "layer: attention must be 0 or 1");
    SA_REQUIRE(d->shift_variant >= 0 && d->shift_variant <= 3, SA_ERR_INVALID, "layer: unknown shift variant");
    const size_t T = (size_t)d->B * d->N, E = (size_t)d->E;
    const int dv = d->E / d->H;
    SA_REQUIRE(T < (size_t)65535 * 8, SA_ERR_SHAPE, "layer: too many tokens for one call");
    size_t off = 0;
    L->codes8 = off; off += up(T * E);
    L->q = off; off += up(T * E * 4);
    L->k = off; off += up(T * E * 4);
    L->v = off; off += up(T * E * 4);
    const size_t code_bytes = up(T * d->H * (d->nbits / 64) * 8);
    L->qc = off; off += code_bytes;
    L->kc = off; off += code_bytes;
    L->kv = off;
    L->attn_ws_bytes = 0;
    if (d->attention == 0) {
        off += up((size_t)d->B * d->H * d->nbits * dv * 4);
        L->attn_ws_bytes = sa_additive_attention_workspace_bytes(d->B, d->H, d->N, d->nbits, dv);
    }
    L->attn_ws = off; off += up(L->attn_ws_bytes);
    L->shift_ws_bytes = sa_shift_mlp_workspace_bytes((long)T, d->E, d->hid);
    L->shift_ws = off; off += up(L->shift_ws_bytes);
    const size_t lin_qkv = sa_shift_linear_workspace_bytes((long)T, d->E, 3 * d->E, d->shift_variant);
    const size_t lin_o = sa_shift_linear_workspace_bytes((long)T, d->E, d->E, d->shift_variant);
    L->lin_ws_bytes = lin_qkv > lin_o ? lin_qkv : lin_o;
    L->lin_ws = off; off += up(L->lin_ws_bytes);
    L->xh = L->logits = L->perm = L->expert_of = L->counts = L->gate = L->disp_ws = L->mult_ws = off;
    L->disp_ws_bytes = L->mult_ws_bytes = 0;
    if (d->moe) {
        L->xh = off; off += up(T * E * 2);
        L->logits = off; off += up(T * 2 * 4);
        L->perm = off; off += up(T * 4);
        L->expert_of = off; off += up(T * 4);
        L->counts = off; off += 256;
        L->gate = off; off += up(T * 4);
        L->disp_ws_bytes = sa_moe_dispatch_workspace_bytes((long)T, 2);
        L->disp_ws = off; off += up(L->disp_ws_bytes);
        L->mult_ws_bytes = sa_mult_mlp_workspace_bytes((long)T, d->E, d->hid);
        L->mult_ws = off; off += up(L->mult_ws_bytes);
    }
    L->needed = L->few = off;
    const size_t few = sa::plan_few_rows((long)T, d->E, d->hid, d->moe != 0, true).bytes;
    off += up(few);
    L->few_wo = off;
    if (few > 0 && d->shift_variant != SA_VARIANT_MFMA_PREPARED) off += up(2 * E * E);      // planes of wo
    L->total = off;
    return SA_OK;
}

}  // namespace

extern "C" size_t sa_layer_workspace_bytes(const sa_layer_desc *desc) {
    LayerLayout L;
    if (plan_layer(desc, &L) != SA_OK) return 0;
    return L.total;
}

extern "C" int sa_layer_forward(const sa_layer_desc *d, void *stream) {
    sa::clear_error();
    LayerLayout L;
    int rc = plan_layer(d, &L);
    if (rc != SA_OK) return rc;
    SA_REQUIRE(d->x && d->y && d->gamma1 && d->beta1 && d->gamma2 && d->beta2 && d->wqkv && d->wo && d->w1 && d->w2 &&
                   d->lut,
               SA_ERR_INVALID, "layer: x, y, the LayerNorm parameters, wqkv, wo, w1, w2 and lut are required");
    if (d->moe) SA_REQUIRE(d->wg && d->bg && d->mw1 && d->mw2, SA_ERR_INVALID, "layer: wg, bg, mw1, mw2 are required");
    SA_REQUIRE(d->workspace != nullptr && d->workspace_bytes >= L.needed, SA_ERR_WORKSPACE,
               "layer: workspace of %zu bytes asked for, %zu needed, %zu given", L.total, L.needed, d->workspace_bytes);
    SA_REQUIRE(sa::aligned16(d->workspace), SA_ERR_ALIGN, "layer: workspace must be 16-byte aligned");
    uint8_t *ws = static_cast<uint8_t *>(d->workspace);
    const long T = (long)d->B * d->N;
    const int E = d->E, dv = d->E / d->H;
    int8_t *codes8 = reinterpret_cast<int8_t *>(ws + L.codes8);
    float *q = reinterpret_cast<float *>(ws + L.q), *k = reinterpret_cast<float *>(ws + L.k);
    float *v = reinterpret_cast<float *>(ws + L.v);
    float *o = q;                                 // Q is dead once it is hashed
    uint64_t *qc = reinterpret_cast<uint64_t *>(ws + L.qc), *kc = reinterpret_cast<uint64_t *>(ws + L.kc);
    float *kv = reinterpret_cast<float *>(ws + L.kv);
    const bool moe = d->moe != 0;
    void *xh = moe ? static_cast<void *>(ws + L.xh) : nullptr;
    float *logits = moe ? reinterpret_cast<float *>(ws + L.logits) : nullptr;
    int32_t *perm = reinterpret_cast<int32_t *>(ws + L.perm);
    int32_t *expert_of = reinterpret_cast<int32_t *>(ws + L.expert_of);
    int32_t *counts = reinterpret_cast<int32_t *>(ws + L.counts);
    float *gate = reinterpret_cast<float *>(ws + L.gate);
    // Sign hash (no projection): the code bits are the signs of the Q and K accumulators, taken in the epilogue of
    // the projection, so Q and K never exist as floats.  Otherwise Q, K, V leave as fp32 and Q, K are hashed.
    const bool fused_hash = d->proj == nullptr && d->nbits == dv && (dv == 64 || dv == 128) && E % 128 == 0 &&
                            d->shift_variant != SA_VARIANT_VALU && d->qkv_scale > 0.0f &&
                            d->qkv_scale - d->qkv_scale == 0.0f;

    // Every step's arguments are checked before the first launch.
    rc = sa::check_layernorm(d->x, T, E, d->gamma1, d->beta1, nullptr, codes8, nullptr, nullptr, nullptr, 0, nullptr);
    if (rc == SA_OK)
        rc = fused_hash ? sa::check_shift_linear_qkv_codes(codes8, d->wqkv, d->B, d->N, d->H, E, d->shift_variant, d->qkv_scale, qc, kc, v,
                                                           ws + L.lin_ws, L.lin_ws_bytes)
                        : sa::check_shift_linear_f32(codes8, d->wqkv, T, E, 3 * E, d->shift_variant, nullptr, 3, q, k, v, ws + L.lin_ws,
                                                     L.lin_ws_bytes);
    if (rc == SA_OK && !fused_hash) rc = sa::check_binarize_pair(q, k, d->B, d->N, d->H, dv, d->proj, d->nbits, qc, kc);
    if (rc == SA_OK)
        rc = d->attention == 0 ? sa::check_additive_attention(qc, kc, v, o, d->B, d->H, d->N, d->N, d->nbits, dv, kv, 3, ws + L.attn_ws,
                                                              L.attn_ws_bytes)
                               : sa::check_hamming_attention(qc, kc, v, nullptr, d->B, d->H, d->N, d->N, d->nbits, dv, d->attn_scale,
                                                             nullptr, codes8, nullptr, SA_VARIANT_AUTO);
    if (rc == SA_OK)
        rc = sa::check_shift_linear_f32(codes8, d->wo, T, E, E, d->shift_variant, d->x, 1, d->y, nullptr, nullptr, ws + L.lin_ws,
                                        L.lin_ws_bytes);
    if (rc == SA_OK)
        rc = sa::check_layernorm(d->y, T, E, d->gamma2, d->beta2, nullptr, codes8, xh, moe ? d->wg : nullptr, moe ? d->bg : nullptr,
                                 moe ? 2 : 0, logits);
    if (rc == SA_OK) rc = check_mlp(*d, E, T);
    if (rc == SA_OK && moe)
        rc = sa::check_moe_dispatch(logits, T, 2, perm, expert_of, counts, gate, ws + L.disp_ws, L.disp_ws_bytes);
    if (rc != SA_OK) return rc;

    // attention half: X_attn = Attn(LayerNorm(X)) + X, left in y.  Narrow rows are normalised by the projection's workgroups.
    const bool norms = !fused_hash && d->shift_variant == SA_VARIANT_MFMA_PREPARED;
    const bool norm_hash = norms && d->proj && sa::norm_hash_one_launch(T, E, d->H, d->nbits);
    const bool packed = d->shift_variant == SA_VARIANT_MFMA || d->shift_variant == SA_VARIANT_AUTO;
    const bool linear_hash = !fused_hash && !norm_hash && (norms || packed) && d->proj && sa::linear_hash_one_launch(T, E, d->H, d->nbits, packed);
    const bool norm_linear = norm_hash || (norms && !linear_hash && sa::norm_linear_one_launch(T, E));
    const sa::FewRowsPlan plan = few_rows(*d, E, T, true, L.total);
    const bool few = plan.bytes > 0;
    sa::ZeroWork zero;                            // for the launch of the MLP half: by the layer's first launch
    if (few) zero = {reinterpret_cast<uint32_t *>(ws + L.few), (int)(plan.ticket_bytes / 4)};
    if (!norm_linear) {
        rc = sa::launch_layernorm(d->x, T, E, d->gamma1, d->beta1, d->eps, d->ln_inv_scale, nullptr, codes8, nullptr, nullptr,
                                  nullptr, 0, nullptr, zero, sa::as_stream(stream));
        if (rc != SA_OK) return rc;
    }
    sa::SideWork side;
    const ShiftWeights weights(*d, E, T, ws + L.shift_ws, &side.decode);
    const int8_t *wo_planes = reinterpret_cast<const int8_t *>(d->wo);
    if (few && packed) {
        sa::add_decode(&side.decode, d->wo, E, E, ws + L.few_wo);
        wo_planes = reinterpret_cast<const int8_t *>(ws + L.few_wo);
    }
    if (fused_hash) {
        if (side.any()) rc = sa::launch_decode_work(side.decode, sa::as_stream(stream));
        if (rc != SA_OK) return rc;
        rc = sa_shift_linear_qkv_codes(codes8, d->wqkv, d->B, d->N, d->H, E, d->shift_variant, d->qkv_scale, qc, kc, v,
                                       ws + L.lin_ws, L.lin_ws_bytes, stream);
        if (rc != SA_OK) return rc;
    } else {
        if (norm_linear) {
            sa::NormRows norm;
            norm.x = d->x;
            norm.gamma = d->gamma1;
            norm.beta = d->beta1;
            norm.eps = d->eps;
            norm.inv_scale = d->ln_inv_scale;
            norm.zero = zero;
            if (norm_hash)
                rc = sa::launch_norm_hash(norm, d->B, d->N, d->H, E, reinterpret_cast<const int8_t *>(d->wqkv), d->qkv_scale, d->proj, d->nbits,
                                          q, k, qc, kc, v, sa::as_stream(stream));
            else
                rc = sa::launch_norm_linear(norm, T, E, reinterpret_cast<const int8_t *>(d->wqkv), d->qkv_scale, q, k, v, sa::as_stream(stream));
        } else if (linear_hash) {
            const uint8_t *planes = d->wqkv;
            if (packed) {                                    // decoded with the MLP's, which otherwise ride in the hash's launch
                sa::DecodeWork wqkv;
                sa::add_decode(&wqkv, d->wqkv, E, 3 * E, ws + L.lin_ws);
                rc = sa::launch_decode_work(side.decode, wqkv, sa::as_stream(stream));
                if (rc != SA_OK) return rc;
                planes = ws + L.lin_ws;
            }
            rc = sa::launch_linear_hash(codes8, d->B, d->N, d->H, E, reinterpret_cast<const int8_t *>(planes), d->qkv_scale, d->proj, d->nbits,
                                        q, k, qc, kc, v, sa::as_stream(stream));
        } else {
            rc = sa_shift_linear_f32(codes8, d->wqkv, T, E, 3 * E, d->shift_variant, d->qkv_scale, nullptr, 3, q, k, v,
                                     ws + L.lin_ws, L.lin_ws_bytes, stream);
        }
        if (rc == SA_OK && !norm_hash && !linear_hash) rc = hash_and_side(q, k, d->B, d->N, d->H, dv, d->proj, d->nbits, qc, kc, side, stream);
        if (rc != SA_OK) return rc;
    }
    if (d->attention == 0) {
        // only the int8 form of the attention output is read (by the output projection): no fp32 write
        rc = sa::additive_attention_fused(qc, kc, v, o, false, d->B, d->H, d->N, d->nbits, dv, d->attn_scale, kv, codes8, nullptr,
                                          d->act_inv_scale, ws + L.attn_ws, L.attn_ws_bytes, stream);
    } else {
        rc = sa_hamming_attention_fused(qc, kc, v, nullptr, d->B, d->H, d->N, d->N, d->nbits, dv, d->attn_scale, nullptr,
                                         codes8, nullptr, d->act_inv_scale, SA_VARIANT_AUTO, stream);
    }
    if (rc != SA_OK) return rc;

    // MLP half: y += MLP(LayerNorm(y)); every row is read by the LayerNorm before an expert adds to it.  Where the MLP is one
    // launch its workgroups normalise their rows themselves, and with prepared weights they make them as well.
    const sa_rows all{nullptr, nullptr, 0, T};
    sa::RowSel sel;
    rc = sa::validate_rows(&all, &sel);
    if (rc != SA_OK) return rc;
    const bool one_launch = !moe && weights.variant == SA_VARIANT_MFMA_PREPARED && sa::shift_mlp_one_launch(sel, E, d->hid, sa::kMlpInLayer);
    const bool project = one_launch && d->shift_variant == SA_VARIANT_MFMA_PREPARED;
    sa::NormRows norm;
    norm.x = norm.out = d->y;
    norm.gamma = d->gamma2;
    norm.beta = d->beta2;
    norm.eps = d->eps;
    norm.inv_scale = d->ln_inv_scale;
    norm.residual = d->x;
    norm.scale = d->o_scale;
    if (few) {
        norm.wo = wo_planes;
        return sa::launch_few_rows({codes8, nullptr, &norm, moe ? d->wg : nullptr, moe ? d->bg : nullptr, nullptr, T, E, d->hid,
                                    reinterpret_cast<const int8_t *>(weights.w1), reinterpret_cast<const int8_t *>(weights.w2), d->lut,
                                    moe ? d->mw1 : nullptr, moe ? d->mw2 : nullptr, d->requant_scale, d->out_scale, d->y, ws + L.few}, plan, sa::as_stream(stream));
    }
    const bool linear_norm = !one_launch && d->shift_variant == SA_VARIANT_MFMA_PREPARED && sa::linear_norm_one_launch(T, E);
    if (project || linear_norm) norm.wo = reinterpret_cast<const int8_t *>(d->wo);
    if (!norm.wo) {
        rc = sa_shift_linear_f32(codes8, d->wo, T, E, E, d->shift_variant, d->o_scale, d->x, 1, d->y, nullptr, nullptr,
                                 ws + L.lin_ws, L.lin_ws_bytes, stream);
        if (rc != SA_OK) return rc;
    }
    if (one_launch) {
        sa::Epilogue e;
        e.yf = d->y;
        e.out_scale = d->out_scale;
        e.accumulate = true;
        return sa::launch_shift_mlp(codes8, &norm, sel, E, d->hid, reinterpret_cast<const int8_t *>(weights.w1),
                                    reinterpret_cast<const int8_t *>(weights.w2), d->lut, d->requant_scale, e, sa::as_stream(stream));
    }
    if (linear_norm)
        rc = sa::launch_linear_norm(codes8, norm, T, E, {codes8, xh, d->wg, d->bg, logits}, sa::as_stream(stream));
    else
        rc = sa_layernorm_quant(d->y, T, E, d->gamma2, d->beta2, d->eps, d->ln_inv_scale, nullptr, codes8, xh,
                                moe ? d->wg : nullptr, moe ? d->bg : nullptr, moe ? 2 : 0, logits, stream);
    if (rc != SA_OK) return rc;
    if (!moe) {
        return sa_shift_mlp(codes8, &all, E, d->hid, weights.w1, weights.w2, d->requant_scale, d->lut, nullptr, d->y, nullptr,
                            d->out_scale, weights.variant, 3 | SA_MLP_ACCUMULATE, ws + L.shift_ws, L.shift_ws_bytes,
                            stream);
    }
    rc = sa_moe_dispatch(logits, T, 2, perm, expert_of, counts, gate, ws + L.disp_ws, L.disp_ws_bytes, stream);
    if (rc != SA_OK) return rc;
    // the experts add to disjoint rows of y
    return experts(*d, weights, codes8, xh, E, T, perm, counts, gate, SA_MLP_ACCUMULATE, ws + L.mult_ws, L.mult_ws_bytes,
                   ws + L.shift_ws, L.shift_ws_bytes, stream);
}
