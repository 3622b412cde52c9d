// LayerNorm of Eq. 2 fused with what its consumers read: the int8 codes of the shift Linears
// (static per-tensor scale), the fp16 rows of the Mult expert and the router logits (Sec. 4.2).
//
// LPR lanes own one row, held in registers (CH float4 per lane), so x is read once: mean, then the
// centred sum of squares (two passes over registers, no E[x^2] - mean^2 cancellation), then the outputs.
// Rows of up to 256 elements take as many lanes as they have float4s (16 to 64), several rows to a
// wavefront.
//
// What bounds it: HBM, 4 B in and 1 (+2, +4) B out per element, once enough rows are in flight: the next row
// of a wavefront is loaded before the sums of the current one, and the sums go through the vector ALU's own
// lane exchanges (a sum over 64 lanes through LDS shuffles is some 400 cycles, four of them in a row's chain).
// int8 codes only, one wavefront per row and no row ahead -> now: 25088 x 64 13.5 -> 5.0 us, 16384 x 256 12.1 -> 8.2,
// 12608 x 768 13.7 -> 12.9 (3.8 TB/s); codes, fp16 rows and router logits: 12608 x 768 19.4 -> 17.9, 50000 x 128
// 25.9 -> 14.5, 131072 x 256 61.5 -> 52.5.
#include "common.h"
#include "gemm_common.h"
#include "layernorm.h"

namespace {

using namespace sa;

typedef _Float16 v4h_t __attribute__((ext_vector_type(4)));

constexpr int kWavesPerBlock = 4;

struct LnArgs {
    const float *x;
    long T;
    int E;
    const float *gamma, *beta;
    float eps, inv_scale;
    float *ln;          // optional outputs
    int8_t *q;
    _Float16 *xh;
    const float *wg;    // [E, n_exp] or null
    const float *bg;    // [n_exp]
    int n_exp;
    float *logits;      // [T, n_exp]
    ZeroWork zero;
};

// ROUTE2: the router has two experts and its weight columns live in registers next to gamma and
// beta (all three depend on the column only), so a wavefront that walks over several rows loads
// them once.  More experts take the weights from memory (the table is small and stays in cache).
template <int LPR, int CH, bool ROUTE2>
__global__ __launch_bounds__(64 * kWavesPerBlock) void layernorm_kernel(LnArgs a, int rows_per_group) {
    constexpr int GROUPS = 64 / LPR;              // rows side by side in a wavefront
    const int lane = threadIdx.x & 63, l = lane % LPR;
    const int E = a.E;
    if (blockIdx.x == 0) zero_words(a.zero);
    // a wavefront walks GROUPS consecutive rows at a time
    const long t0 = ((long)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6)) * rows_per_group * GROUPS + lane / LPR;
    if (t0 - lane / LPR >= a.T) return;
    constexpr bool CACHE = CH <= 8;               // wider rows re-read gamma and beta per row (registers)
    constexpr int PC = CACHE ? CH : 1;
    auto load_row = [&](long t, float4 (&v)[CH]) {
        const float *row = a.x + (size_t)(t < a.T ? t : a.T - 1) * E;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int j = (c * LPR + l) * 4;
            v[c] = j < E ? *reinterpret_cast<const float4 *>(row + j) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    };
    constexpr bool AHEAD = CH <= 4;               // the next row in flight (registers)
    float4 nxt[AHEAD ? CH : 1];
    if constexpr (AHEAD) load_row(t0, nxt);
    float4 gm[PC], bt[PC], w0[PC], w1[PC];
#pragma unroll
    for (int c = 0; c < PC; ++c) {
        const int j = (c * LPR + l) * 4;
        const bool in = j < E;
        gm[c] = in ? *reinterpret_cast<const float4 *>(a.gamma + j) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        bt[c] = in ? *reinterpret_cast<const float4 *>(a.beta + j) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (ROUTE2) {                             // wg rows j..j+3: (e0, e1) pairs
            w0[c] = in ? *reinterpret_cast<const float4 *>(a.wg + 2 * j) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            w1[c] = in ? *reinterpret_cast<const float4 *>(a.wg + 2 * j + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    }
    for (int it = 0; it < rows_per_group; ++it) {
        const long t = t0 + (long)it * GROUPS;
        if (t - lane / LPR >= a.T) return;        // the whole wavefront is past the end
        const bool row_ok = t < a.T;
        float4 v[CH];
        if constexpr (AHEAD) {
#pragma unroll
            for (int c = 0; c < CH; ++c) v[c] = nxt[c];
            if (it + 1 < rows_per_group) load_row(t + GROUPS, nxt);
        } else {
            load_row(t, v);
        }
        float mean, rstd;
        row_stats<LPR, CH>(v, l, E, a.eps, mean, rstd);
        float part[kMaxExperts];
#pragma unroll
        for (int e = 0; e < kMaxExperts; ++e) part[e] = 0.0f;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int j = (c * LPR + l) * 4;
            if (j >= E) continue;
            const float4 g = CACHE ? gm[CACHE ? c : 0] : *reinterpret_cast<const float4 *>(a.gamma + j);
            const float4 b = CACHE ? bt[CACHE ? c : 0] : *reinterpret_cast<const float4 *>(a.beta + j);
            float y[4];
            normalise(v[c], mean, rstd, g, b, y);
            if (row_ok) {
                const size_t o = (size_t)t * E + j;
                if (a.ln) *reinterpret_cast<float4 *>(a.ln + o) = make_float4(y[0], y[1], y[2], y[3]);
                if (a.q) *reinterpret_cast<uint32_t *>(a.q + o) = codes_of(y, a.inv_scale);
                if (a.xh) {
                    v4h_t h;
#pragma unroll
                    for (int i = 0; i < 4; ++i) h[i] = (_Float16)y[i];
                    *reinterpret_cast<v4h_t *>(a.xh + o) = h;
                }
            }
            if (ROUTE2 && CACHE) {
                part[0] = __builtin_fmaf(y[0], w0[c].x, part[0]);
                part[1] = __builtin_fmaf(y[0], w0[c].y, part[1]);
                part[0] = __builtin_fmaf(y[1], w0[c].z, part[0]);
                part[1] = __builtin_fmaf(y[1], w0[c].w, part[1]);
                part[0] = __builtin_fmaf(y[2], w1[c].x, part[0]);
                part[1] = __builtin_fmaf(y[2], w1[c].y, part[1]);
                part[0] = __builtin_fmaf(y[3], w1[c].z, part[0]);
                part[1] = __builtin_fmaf(y[3], w1[c].w, part[1]);
            } else if (a.logits) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int e = 0; e < kMaxExperts; ++e)
                        if (e < a.n_exp) part[e] = __builtin_fmaf(y[i], a.wg[(size_t)(j + i) * a.n_exp + e], part[e]);
            }
        }
        if (a.logits) {
#pragma unroll
            for (int e = 0; e < kMaxExperts; ++e) {
                if (e >= a.n_exp) break;
                const float sum = group_sum<LPR>(part[e]);
                if (l == 0 && row_ok) a.logits[(size_t)t * a.n_exp + e] = sum + a.bg[e];
            }
        }
    }
}

template <int LPR, int CH>
int launch(const LnArgs &a, hipStream_t st) {
    // up to four rows per lane group amortise the per-column parameters; keep >= 4096 wavefronts (16 per CU) in flight
    constexpr int GROUPS = 64 / LPR;
    const long steps = (a.T + GROUPS - 1) / GROUPS;
    int rows_per_group = 1;
    while (rows_per_group < 4 && steps / (2 * rows_per_group) >= 4096) rows_per_group *= 2;
    const long waves = (steps + rows_per_group - 1) / rows_per_group;
    const long blocks = (waves + kWavesPerBlock - 1) / kWavesPerBlock;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_layernorm_quant: too many rows");
    const dim3 grid((unsigned)blocks), block(64 * kWavesPerBlock);
    if (a.logits && a.n_exp == 2 && CH <= 8)
        layernorm_kernel<LPR, CH, true><<<grid, block, 0, st>>>(a, rows_per_group);
    else
        layernorm_kernel<LPR, CH, false><<<grid, block, 0, st>>>(a, rows_per_group);
    return check_launch("sa_layernorm_quant");
}

}  // namespace

// Everything sa_layernorm_quant asks of its arguments.
int sa::check_layernorm(const float *x, long T, int E, const float *gamma, const float *beta, const float *ln_or_null,
                        const int8_t *q_or_null, const void *xh_or_null, const float *wg_or_null, const float *bg_or_null, int n_experts,
                        const float *logits_or_null) {
    SA_REQUIRE(T >= 0 && E > 0, SA_ERR_INVALID, "sa_layernorm_quant: T < 0 or E <= 0");
    SA_REQUIRE(E % 4 == 0, SA_ERR_SHAPE, "sa_layernorm_quant: E (%d) must be a multiple of 4", E);
    SA_REQUIRE(E <= 8192, SA_ERR_UNSUPPORTED, "sa_layernorm_quant: rows of more than 8192 elements are not built");
    const bool route = logits_or_null != nullptr;
    if (route) {
        SA_REQUIRE(wg_or_null && bg_or_null, SA_ERR_INVALID, "sa_layernorm_quant: logits need wg and bg");
        SA_REQUIRE(n_experts >= 2 && n_experts <= kMaxExperts, SA_ERR_SHAPE,
                   "sa_layernorm_quant: 2 to 8 experts (got %d)", n_experts);
    }
    if (T == 0) return SA_OK;
    SA_REQUIRE(x && gamma && beta, SA_ERR_INVALID, "sa_layernorm_quant: NULL buffer");
    SA_REQUIRE(ln_or_null || q_or_null || xh_or_null || route, SA_ERR_INVALID, "sa_layernorm_quant: no output requested");
    SA_REQUIRE(sa::aligned16(x) && sa::aligned16(gamma) && sa::aligned16(beta) && sa::aligned16(ln_or_null) &&
                   sa::aligned16(q_or_null) && sa::aligned16(xh_or_null) && sa::aligned16(wg_or_null) &&
                   sa::aligned16(bg_or_null) && sa::aligned16(logits_or_null),
               SA_ERR_ALIGN, "sa_layernorm_quant: pointers must be 16-byte aligned");
    return SA_OK;
}

extern "C" int sa_layernorm_quant(const float *x, long T, int E, const float *gamma, const float *beta, float eps,
                                  float inv_scale, float *ln_or_null, int8_t *q_or_null, void *xh_or_null,
                                  const float *wg_or_null, const float *bg_or_null, int n_experts,
                                  float *logits_or_null, void *stream) {
    sa::clear_error();
    const int bad = sa::check_layernorm(x, T, E, gamma, beta, ln_or_null, q_or_null, xh_or_null, wg_or_null, bg_or_null, n_experts,
                                        logits_or_null);
    if (bad != SA_OK || T == 0) return bad;
    return sa::launch_layernorm(x, T, E, gamma, beta, eps, inv_scale, ln_or_null, q_or_null, xh_or_null, wg_or_null, bg_or_null, n_experts,
                                logits_or_null, sa::ZeroWork(), sa::as_stream(stream));
}

int sa::launch_layernorm(const float *x, long T, int E, const float *gamma, const float *beta, float eps, float inv_scale, float *ln, int8_t *q,
                         void *xh, const float *wg, const float *bg, int n_experts, float *logits, const ZeroWork &zero, hipStream_t st) {
    const bool route = logits != nullptr;
    const LnArgs a{x, T, E, gamma, beta, eps, inv_scale, ln, q, static_cast<_Float16 *>(xh),
                   route ? wg : nullptr, route ? bg : nullptr, route ? n_experts : 0, logits, zero};
    const int ch = (E + 255) / 256;
    if (E <= 64) return launch<16, 1>(a, st);
    if (E <= 128) return launch<32, 1>(a, st);
    if (ch <= 1) return launch<64, 1>(a, st);
    if (ch <= 2) return launch<64, 2>(a, st);
    if (ch <= 3) return launch<64, 3>(a, st);
    if (ch <= 4) return launch<64, 4>(a, st);
    if (ch <= 8) return launch<64, 8>(a, st);
    if (ch <= 16) return launch<64, 16>(a, st);
    return launch<64, 32>(a, st);
}
