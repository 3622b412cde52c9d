// sa_additive_attention: K^T V and Q (K^T V) as Add layers (Eq. 3, O_Add; Sec. 4.1,
// MatMul order exchanged to Q(KV); appendix: the scale is multiplied after the adds).
//
// Both kernels are sign-select-and-accumulate on the vector ALU: the operand
// that every lane shares (a row of V, a row of K^T V) arrives through scalar
// loads and is consumed straight from scalar registers; the sign each lane
// applies comes from its own code bit.  acc = fma(+-1.0f, v, acc) is an exact
// add or subtract (the product never rounds) and issues at the rate of v_add.
//
//   K^T V   : lane j  <-> code bit j of one 64-bit word, accumulators = the dv
//             columns of row j; tokens stream by, split over wavefronts and
//             workgroups, partial sums meet in LDS and then in a second pass,
//             always in the same order.
//   Q(K^T V): lane n  <-> token n, accumulators = the dv outputs of the token.
#include <utility>

#include "common.h"

namespace {

using sa::kWave;

constexpr int kKtvWaves = 4;   // wavefronts per workgroup that share one (b, h, word)

template <int DV, bool ZO>
__global__ __launch_bounds__(256) void ktv_kernel(const uint64_t *__restrict__ k_codes,
                                                  const float *__restrict__ v,
                                                  float *__restrict__ dst, int H, int Nk, int W,
                                                  int splits, int tokens_per_wave) {
    __shared__ float red[kWave * DV];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // blockIdx.x = (bh * W + w) * splits + split
    const int split = blockIdx.x % splits;
    const long bhw = blockIdx.x / splits;
    const int w = (int)(bhw % W);
    const long bh = bhw / W;
    const int b = (int)(bh / H), h = (int)(bh % H);

    float acc[DV];
#pragma unroll
    for (int c = 0; c < DV; ++c) acc[c] = 0.0f;

    const long first = ((long)split * kKtvWaves + wave) * tokens_per_wave;
    const long last = min((long)Nk, first + tokens_per_wave);
    for (long n = first; n < last; ++n) {
        const uint64_t word = k_codes[((size_t)bh * Nk + n) * W + w];           // uniform
        const float *vr = v + (((size_t)b * Nk + n) * H + h) * DV;              // uniform
        const float sig = ((word >> lane) & 1ull) ? 1.0f : (ZO ? 0.0f : -1.0f);
#pragma unroll
        for (int c = 0; c < DV; ++c) acc[c] = __builtin_fmaf(sig, vr[c], acc[c]);
    }

    // cross-wavefront reduction through LDS, fixed order ((w0 + w1) + w2) + w3
    for (int s = 1; s < kKtvWaves; ++s) {
        if (wave == s) {
#pragma unroll
            for (int c = 0; c < DV; ++c) red[c * kWave + lane] = acc[c];
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int c = 0; c < DV; ++c) acc[c] += red[c * kWave + lane];
        }
        __syncthreads();
    }
    if (wave == 0) {
        // dst: [splits][BH][nbits][DV]; row = w*64 + lane
        const size_t BH_rows = (size_t)gridDim.x / splits * 64;   // BH * W * 64 = BH * nbits
        float *o = dst + ((size_t)split * BH_rows + (size_t)bhw * 64 + lane) * DV;
#pragma unroll
        for (int c = 0; c < DV; c += 4)
            *reinterpret_cast<float4 *>(o + c) = make_float4(acc[c], acc[c + 1], acc[c + 2], acc[c + 3]);
    }
}

template <int DV, bool ZO>
__global__ __launch_bounds__(256) void qkv_kernel(const uint64_t *__restrict__ q_codes,
                                                  const float *__restrict__ kv,
                                                  float *__restrict__ out, int H, int Nq, int W,
                                                  int n_chunks, long n_tasks, float scale,
                                                  const int32_t *__restrict__ den, float eps) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long task = (long)blockIdx.x * (blockDim.x >> 6) + wave;
    if (task >= n_tasks) return;
    const int chunk = (int)(task % n_chunks);
    const long bh = task / n_chunks;
    const int b = (int)(bh / H), h = (int)(bh % H);
    const int n = chunk * 64 + lane;
    const int n_ld = min(n, Nq - 1);

    float acc[DV];
#pragma unroll
    for (int c = 0; c < DV; ++c) acc[c] = 0.0f;

    const uint64_t *code = q_codes + ((size_t)bh * Nq + n_ld) * W;
    const float *kv_bh = kv + (size_t)bh * W * 64 * DV;
    for (int w = 0; w < W; ++w) {
        const uint64_t word = ~code[w];
        const uint32_t half[2] = {(uint32_t)word, (uint32_t)(word >> 32)};
#pragma unroll
        for (int j = 0; j < 64; ++j) {
            // bit 1 -> +1.0f, bit 0 -> -1.0f: move the inverted bit into the float sign
            // ({0,1} codes: bit 1 -> 1.0f, bit 0 -> 0.0f; `word` is the inverted code)
            const uint32_t s = ZO ? ((~half[j >> 5] >> (j & 31)) & 1u) * 0x3f800000u
                                  : ((half[j >> 5] << (31 - (j & 31))) & 0x80000000u) | 0x3f800000u;
            const float sig = __builtin_bit_cast(float, s);
            const float *row = kv_bh + (size_t)(w * 64 + j) * DV;                // uniform
#pragma unroll
            for (int c = 0; c < DV; ++c) acc[c] = __builtin_fmaf(sig, row[c], acc[c]);
        }
    }
    if (n < Nq) {
        float *o = out + (((size_t)b * Nq + n) * H + h) * DV;
        const float f = den ? 1.0f / ((float)den[(size_t)bh * Nq + n] + eps) : scale;
#pragma unroll
        for (int c = 0; c < DV; c += 4)
            *reinterpret_cast<float4 *>(o + c) = make_float4(f * acc[c], f * acc[c + 1], f * acc[c + 2], f * acc[c + 3]);
    }
}

// ksum[bh, j] += number of tokens of the block's range whose code bit j is set (lane <-> bit of one word).
// The code words are wave-uniform; eight are fetched before any is used so that their latencies overlap.
__global__ __launch_bounds__(256) void bit_count_kernel(const uint64_t *__restrict__ k_codes, int32_t *__restrict__ ksum,
                                                        int Nk, int W, int splits, int tokens_per_wave) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int split = blockIdx.x % splits;
    const long bhw = blockIdx.x / splits;
    const int w = (int)(bhw % W);
    const long bh = bhw / W;
    const long first = ((long)split * 4 + wave) * tokens_per_wave;
    const long last = min((long)Nk, first + tokens_per_wave);
    const uint64_t *base = k_codes + (size_t)bh * Nk * W + w;
    int32_t cnt = 0;
    long n = first;
    for (; n + 8 <= last; n += 8) {
        uint64_t wd[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) wd[t] = base[(size_t)(n + t) * W];             // uniform
#pragma unroll
        for (int t = 0; t < 8; ++t) cnt += (int32_t)((wd[t] >> lane) & 1ull);
    }
    for (; n < last; ++n) cnt += (int32_t)((base[(size_t)n * W] >> lane) & 1ull);
    if (cnt) atomicAdd(ksum + (size_t)bhw * 64 + lane, cnt);                        // integers: order-independent
}

// den[bh, n] = sum over the set bits j of query n's code of ksum[bh, j]  (thread <-> query).  The sums of every
// 4-bit group over its 16 possible nibbles are tabulated in LDS first (nbits / 4 groups x 16 entries), so a query
// costs one table read per nibble of its code.
__global__ __launch_bounds__(256) void den_kernel(const uint64_t *__restrict__ q_codes, const int32_t *__restrict__ ksum,
                                                  int32_t *__restrict__ den, int Nq, int W, int n_chunks) {
    extern __shared__ int32_t tab[];                 // [W * 16 groups][16]
    const long bh = blockIdx.x / n_chunks;
    const int chunk = blockIdx.x % n_chunks;
    const int n_entries = W * 16 * 16;
    for (int i = threadIdx.x; i < n_entries; i += blockDim.x) {
        const int g = i >> 4, nib = i & 15;
        const int32_t *k4 = ksum + (size_t)bh * W * 64 + g * 4;
        tab[i] = ((nib & 1) ? k4[0] : 0) + ((nib & 2) ? k4[1] : 0) + ((nib & 4) ? k4[2] : 0) + ((nib & 8) ? k4[3] : 0);
    }
    __syncthreads();
    const int n = chunk * 256 + threadIdx.x;
    if (n >= Nq) return;
    const uint64_t *code = q_codes + ((size_t)bh * Nq + n) * W;
    int32_t d = 0;
    for (int w = 0; w < W; ++w) {
        const uint64_t word = code[w];
        const uint32_t half[2] = {(uint32_t)word, (uint32_t)(word >> 32)};
#pragma unroll
        for (int g = 0; g < 16; ++g) d += tab[((w * 16 + g) << 4) + ((half[g >> 3] >> (4 * (g & 7))) & 15u)];
    }
    den[(size_t)bh * Nq + n] = d;
}

// Depthwise 3x3 over the token grid, zero padding.
// A thread computes RY outputs of one column of the token grid, one below the other, for four channels: 3 (RY + 2) neighbours
// instead of 9 RY, all of them asked for before the first is used, the channels' weights in registers.  Lanes run along the
// channels and then the grid, so that every load is whole lines.  The taps of an output are added in their order, those outside
// the grid left out.  i: 4-channel columns of (image, strip of RY rows, x), 32-bit with divisions by multiplication (SMALL), as
// 64-bit divisions took longer than the loads: 32 images of 56 x 56 x 32 15.1 -> 10.4 us with them gone and RY = 4, where the
// bytes (v, and out read and written) take 8.
// LINE: a grid of one row as a column of gw tokens (gh = gw, gw = 1 here), whose taps are those of the kernel's middle row.
template <int RY, bool SMALL, bool LINE>
__global__ __launch_bounds__(256) void dwconv3x3_kernel(const float *__restrict__ v, const float *__restrict__ w,
                                                        const float *__restrict__ bias, float *__restrict__ out, int accumulate,
                                                        long total, int gh, int gw, int E4, int strips, sa::FastDiv by_e4,
                                                        sa::FastDiv by_gw, sa::FastDiv by_strips) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    int c4, x, y0;
    long b;
    if constexpr (SMALL) {
        const uint32_t r = by_e4((uint32_t)i), s = by_gw(r), bb = by_strips(s);
        c4 = (int)((uint32_t)i - r * (uint32_t)E4);
        x = (int)(r - s * (uint32_t)gw);
        y0 = (int)(s - bb * (uint32_t)strips) * RY;
        b = bb;
    } else {
        const long r = i / E4, s = r / gw;
        c4 = (int)(i - r * E4);
        x = (int)(r - s * gw);
        b = s / strips;
        y0 = (int)(s - b * strips) * RY;
    }
    const size_t E = (size_t)E4 * 4, row = (size_t)gw * E;
    const int c = c4 * 4;
    const float *vc = v + ((size_t)b * gh * gw + x) * E + c;          // row 0 of this column
    float *oc = out + ((size_t)b * gh * gw + x) * E + c;
    const bool left = x > 0, right = x + 1 < gw;

    float wt[4][9];                                                    // [channel][tap]
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const float4 t = *reinterpret_cast<const float4 *>(w + (size_t)c * 9 + 4 * q);
        const float tv[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) wt[(4 * q + e) / 9][(4 * q + e) % 9] = tv[e];
    }
    // (rows and columns outside the grid are read at its edge and not used)
    float4 n[RY + 2][3];
#pragma unroll
    for (int r = 0; r < RY + 2; ++r) {
        const float *p = vc + (size_t)min(max(y0 + r - 1, 0), gh - 1) * row;
        if constexpr (!LINE) n[r][0] = *reinterpret_cast<const float4 *>(p - (left ? E : 0));
        n[r][1] = *reinterpret_cast<const float4 *>(p);
        if constexpr (!LINE) n[r][2] = *reinterpret_cast<const float4 *>(p + (right ? E : 0));
    }
    float4 old[RY];
    if (accumulate) {
#pragma unroll
        for (int r = 0; r < RY; ++r) old[r] = *reinterpret_cast<const float4 *>(oc + (size_t)min(y0 + r, gh - 1) * row);
    }
    float start[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) start[q] = bias ? bias[c + q] : 0.0f;
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        if (y0 + r >= gh) break;
        float acc[4] = {start[0], start[1], start[2], start[3]};
#pragma unroll
        for (int t = LINE ? 3 : 0; t < (LINE ? 6 : 9); ++t) {
            const int dy = LINE ? t - 4 : t / 3 - 1, dx = LINE ? 0 : t % 3 - 1;
            const float4 nv = n[r + 1 + dy][dx + 1];
            const bool in = (dy == 0 || (dy < 0 ? y0 + r > 0 : y0 + r + 1 < gh)) && (dx == 0 || (dx < 0 ? left : right));
            const float x4[4] = {nv.x, nv.y, nv.z, nv.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float sum = __builtin_fmaf(wt[q][t], x4[q], acc[q]);
                acc[q] = in ? sum : acc[q];
            }
        }
        float4 o = make_float4(acc[0], acc[1], acc[2], acc[3]);
        if (accumulate) {
            o.x += old[r].x; o.y += old[r].y; o.z += old[r].z; o.w += old[r].w;
        }
        *reinterpret_cast<float4 *>(oc + (size_t)(y0 + r) * row) = o;
    }
}

struct KtvPlan {
    int splits;            // workgroups per (b, h, word)
    int tokens_per_wave;
};

KtvPlan plan_ktv(int B, int H, int Nk, int nbits) {
    const long groups = (long)B * H * (nbits / 64);
    // aim at ~4096 wavefronts in flight, at least 64 tokens per wavefront
    long splits = (1024 + groups - 1) / groups;
    const long max_splits = ((long)Nk + 64 * kKtvWaves - 1) / (64 * kKtvWaves);
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    if (splits > 64) splits = 64;
    const long waves = splits * kKtvWaves;
    KtvPlan p;
    p.splits = (int)splits;
    p.tokens_per_wave = (int)(((long)Nk + waves - 1) / waves);
    if (p.tokens_per_wave < 1) p.tokens_per_wave = 1;
    return p;
}

bool dv_ok(int dv) { return dv == 32 || dv == 64 || dv == 128; }

}  // namespace

extern "C" size_t sa_additive_attention_workspace_bytes(int B, int H, int Nk, int nbits, int dv) {
    if (B <= 0 || H <= 0 || Nk <= 0 || nbits <= 0 || dv <= 0 || nbits % 64) return 0;
    // room for whichever variant runs: partial sums [splits][B*H][nbits][dv]
    const KtvPlan p = plan_ktv(B, H, Nk, nbits);
    int splits = p.splits;
    if (sa::additive_mfma_ktv_supported(nbits, dv)) {
        const sa::AdditiveMfmaPlan m = sa::plan_additive_mfma(B, H, Nk, nbits, dv);
        if (m.splits > splits) splits = m.splits;
    }
    if (splits <= 1) return 0;
    return (size_t)splits * B * H * nbits * dv * sizeof(float);
}

namespace {

// What the two Add layers do beyond the plain call.  zero_one: a clear code bit contributes nothing instead of -V, the
// bit counts are left in ksum (phase 1) or taken from there (phase 2), and rows leave as acc / (normaliser + eps) instead
// of scale * acc.  ksum_part: room for [splits][B*H][nbits] counts; den: room for the normalisers [B*H, Nq].
struct AddMode {
    bool zero_one = false;
    int32_t *ksum = nullptr, *ksum_part = nullptr, *den = nullptr;
    float eps = 0.0f;
    bool want_out = true;             // false: only the forms below are read
    int8_t *xq = nullptr;
    _Float16 *xh = nullptr;
    float act_inv_scale = 0.0f;
};

// ksum by a kernel of its own (what the vector-ALU variant of phase 1 needs beside K^T V).
int count_bits(const uint64_t *k_codes, int32_t *ksum, long BH, int Nk, int nbits, hipStream_t st) {
    int rc = sa::launch_zero(ksum, (size_t)BH * nbits * sizeof(int32_t), st);
    if (rc != SA_OK || Nk == 0) return rc;
    const int W = nbits / 64;
    // about 64 tokens per wavefront (eight batches of eight loads): short dependent chains, many wavefronts
    long splits = ((long)Nk + 255) / 256;
    if (splits > 1024) splits = 1024;
    const int tokens_per_wave = (int)(((long)Nk + splits * 4 - 1) / (splits * 4));
    const long blocks = BH * W * splits;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_linear_attention_01: grid too large");
    bit_count_kernel<<<dim3((unsigned)blocks), dim3(256), 0, st>>>(k_codes, ksum, Nk, W, (int)splits, tokens_per_wave);
    return sa::check_launch("sa_linear_attention_01(bit counts)");
}

// Token splits of phase 1: more than one means as many partials of K^T V in the workspace.
int ktv_splits(bool valu, int B, int H, int Nk, int nbits, int dv) {
    return !valu && sa::additive_mfma_ktv_supported(nbits, dv) ? sa::plan_additive_mfma(B, H, Nk, nbits, dv).splits
                                                               : plan_ktv(B, H, Nk, nbits).splits;
}

}  // namespace

// Everything sa_additive_attention asks of its arguments.
int sa::check_additive_attention(const uint64_t *q_codes, const uint64_t *k_codes, const float *v, const float *out, int B, int H,
                                 int Nq, int Nk, int nbits, int dv, const float *kv, int phases, const void *workspace,
                                 size_t workspace_bytes) {
    SA_REQUIRE(phases >= 1 && phases <= 7 && (phases & 3) != 0, SA_ERR_INVALID,
               "sa_additive_attention: phases must be 1, 2 or 3, optionally + 4");
    const bool valu = (phases & SA_ADDITIVE_VALU) != 0;
    SA_REQUIRE(B >= 0 && H >= 0 && Nq >= 0 && Nk >= 0 && nbits > 0 && dv > 0, SA_ERR_INVALID,
               "sa_additive_attention: negative size");
    SA_REQUIRE(nbits % 64 == 0 && nbits <= 4096, SA_ERR_SHAPE,
               "sa_additive_attention: nbits %d must be a multiple of 64, at most 4096", nbits);
    SA_REQUIRE(dv_ok(dv), SA_ERR_UNSUPPORTED, "sa_additive_attention: dv must be 32, 64 or 128 (got %d)", dv);
    SA_REQUIRE((long)B * H < (1L << 20), SA_ERR_SHAPE, "sa_additive_attention: B*H too large");
    const long BH = (long)B * H;
    if (BH == 0) return SA_OK;
    SA_REQUIRE(kv != nullptr, SA_ERR_INVALID, "sa_additive_attention: kv is NULL");
    SA_REQUIRE(sa::aligned16(q_codes) && sa::aligned16(k_codes) && sa::aligned16(v) &&
                   sa::aligned16(out) && sa::aligned16(kv) && sa::aligned16(workspace),
               SA_ERR_ALIGN, "sa_additive_attention: pointers must be 16-byte aligned");
    if (phases & 2) {
        SA_REQUIRE(Nq == 0 || (q_codes != nullptr && out != nullptr), SA_ERR_INVALID,
                   "sa_additive_attention: phase 2 needs q_codes and out");
        const bool mfma = !valu && additive_mfma_qkv_supported(nbits, dv);
        const long blocks = mfma ? BH * (dv / 32) * (((long)Nq + 255) / 256) : (BH * (((long)Nq + 63) / 64) + 3) / 4;
        SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_additive_attention: grid too large");
    }
    if ((phases & 1) && Nk > 0) {
        SA_REQUIRE(k_codes != nullptr && v != nullptr, SA_ERR_INVALID, "sa_additive_attention: phase 1 needs k_codes and v");
        const int splits = ktv_splits(valu, B, H, Nk, nbits, dv);
        const size_t need = splits > 1 ? (size_t)splits * BH * nbits * dv * sizeof(float) : 0;
        SA_REQUIRE(need == 0 || (workspace != nullptr && workspace_bytes >= need), SA_ERR_WORKSPACE,
                   "sa_additive_attention: workspace of %zu bytes needed, %zu given", need, workspace_bytes);
    }
    return SA_OK;
}

namespace {

int run_additive(const uint64_t *q_codes, const uint64_t *k_codes, const float *v, float *out, int B, int H, int Nq,
                 int Nk, int nbits, int dv, float scale, float *kv, int phases, void *workspace,
                 size_t workspace_bytes, void *stream, const AddMode &mode) {
    const int bad = sa::check_additive_attention(q_codes, k_codes, v, out, B, H, Nq, Nk, nbits, dv, kv, phases, workspace, workspace_bytes);
    const long BH = (long)B * H;
    if (bad != SA_OK || BH == 0) return bad;
    const bool valu = (phases & SA_ADDITIVE_VALU) != 0;
    hipStream_t st = sa::as_stream(stream);
    const int W = nbits / 64;
    const size_t kv_elems = (size_t)BH * nbits * dv;
    const bool qkv_mfma = !valu && sa::additive_mfma_qkv_supported(nbits, dv);
    // What phase 2 reads: K^T V (and the counts), or the partials of phase 1 where it sums them itself.
    sa::AddFused f;
    f.kv_in = kv;
    f.ksum_in = mode.ksum;
    f.scale = scale;
    f.eps = mode.eps;
    f.out = mode.want_out ? out : nullptr;
    f.xq = mode.xq;
    f.xh = mode.xh;
    f.act_inv_scale = mode.act_inv_scale;
    // The convolution that follows {0,1} codes reads and writes them, and reads V: up to 120 MiB of either both are still in the last-level
    // cache (256 MiB) then.  More outputs leave as a stream, which ends the launch sooner than the convolution is held up (hash, attention and
    // convolution, streamed and kept, us: 16 x 4096 tokens x 256 115.6, 108.9; 2 x 16384 x 256 63.3, 61.3; 222 x 196 x 384 124.8, 117.8; 2 x 16384 x 768
    // 215.3, 206.4; 17 x 784 x 256 37.0, 36.5; 445 x 196 x 384, 128 MiB, 236.8, 243.5; 166 x 784 x 384 337.9, 343.4).  So do those of
    // tokens of one line, 32 columns, beyond 8 MiB (32 x 3136 x 32 32.5, 33.4; 9 x 16384 41.1, 42.0; 318 x 784 57.2, 57.5; 47 x 16384 157.1, 158.3; but 31 x
    // 16384 112.7, 111.1).
    f.keep = mode.zero_one && BH * Nq * dv * 4 <= (H * dv >= 64 ? 120L : 8L) << 20;

    if (phases & 1) {
        if (Nk == 0) {
            int rc = sa::launch_zero(kv, kv_elems * sizeof(float), st);   // empty sum
            if (rc == SA_OK && mode.zero_one) rc = sa::launch_zero(mode.ksum, (size_t)BH * nbits * sizeof(int32_t), st);
            if (rc != SA_OK) return rc;
        } else {
            const bool mfma = !valu && sa::additive_mfma_ktv_supported(nbits, dv);
            sa::AdditiveMfmaPlan m{};
            KtvPlan p{};
            if (mfma) m = sa::plan_additive_mfma(B, H, Nk, nbits, dv);
            else p = plan_ktv(B, H, Nk, nbits);
            if (mfma && qkv_mfma && (phases & 2) && Nq > 0 && !mode.zero_one && sa::additive_mfma_one_launch(m, Nq, Nk, nbits))
                return sa::launch_ktv_qkv(k_codes, v, kv, q_codes, f, B, H, Nq, Nk, nbits, dv, st);
            const int splits = mfma ? m.splits : p.splits;
            float *dst = kv;
            int32_t *counts = mode.ksum;
            if (splits > 1) {
                dst = static_cast<float *>(workspace);
                counts = mode.ksum_part;
            }
            int rc;
            if (mfma) {
                rc = sa::launch_ktv_mfma(k_codes, v, dst, counts, B, H, Nk, nbits, dv, m, mode.zero_one, st);
            } else {
                const long blocks = BH * W * p.splits;
                SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_additive_attention: grid too large");
                const dim3 grid((unsigned)blocks), block(kKtvWaves * kWave);
#define SA_KTV(DV_, ZO_) ktv_kernel<DV_, ZO_><<<grid, block, 0, st>>>(k_codes, v, dst, H, Nk, W, p.splits, p.tokens_per_wave)
                switch (dv) {
                    case 32: if (mode.zero_one) SA_KTV(32, true); else SA_KTV(32, false); break;
                    case 64: if (mode.zero_one) SA_KTV(64, true); else SA_KTV(64, false); break;
                    default: if (mode.zero_one) SA_KTV(128, true); else SA_KTV(128, false); break;
                }
#undef SA_KTV
                rc = sa::check_launch("sa_additive_attention(K^T V)");
                if (rc == SA_OK && mode.zero_one) rc = count_bits(k_codes, mode.ksum, BH, Nk, nbits, st);
            }
            if (rc != SA_OK) return rc;
            if (splits > 1) {
                if (mfma && qkv_mfma && (phases & 2) && Nq > 0 && sa::additive_mfma_sums_partials(splits, nbits, dv)) {
                    f.kv_in = dst;
                    f.kv_out = kv;
                    f.ksum_in = counts;
                    f.ksum_out = mode.ksum;
                    f.splits = splits;
                } else {
                    rc = sa::launch_ktv_sum(dst, kv, mfma && mode.zero_one ? counts : nullptr, mode.ksum, BH, nbits, dv, splits, st);
                    if (rc != SA_OK) return rc;
                }
            }
        }
    }
    if ((phases & 2) && Nq > 0) {
        // Made just before its stores, a row's address lets the wavefronts of a CU take turns row by row, all at the same rows of tiles that lie
        // a power of two apart.  As long as the caches take the outputs that costs nothing; beyond, memory falls behind, by how the card's
        // pages lie (both products on three cards, us, as the compiler makes them, just before and ahead: 6 x 6482 tokens x 4 heads x 64 bits x 64 27.9; 31.7, 27.8, 25.7; 26.5, 8 x 16384 63.8; 69.6, 64.6, 61.1; 61.9;
        // 16 MiB of outputs, 1 x 16384, 18.0; 16.6, 16.6, 16.3; 16.7, 64 x 784 x 2 heads x 32 15.4; 14.0; 14.6).
        const long row_bytes = (f.out ? 4 : 0) + (f.xq ? 1 : 0) + (f.xh ? 2 : 0);
        f.rows_ahead = BH * Nq * dv * row_bytes > 24L << 20;
        if (qkv_mfma) return sa::launch_qkv_mfma(q_codes, f, B, H, Nq, nbits, dv, mode.zero_one, st);
        const int32_t *den = nullptr;
        if (mode.zero_one) {
            const int den_chunks = (Nq + 255) / 256;
            const long blocks = BH * den_chunks;
            SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_linear_attention_01: grid too large");
            den_kernel<<<dim3((unsigned)blocks), dim3(256), (size_t)nbits * 4 * sizeof(int32_t), st>>>(q_codes, mode.ksum, mode.den, Nq,
                                                                                                      W, den_chunks);
            int rc = sa::check_launch("sa_linear_attention_01(normaliser)");
            if (rc != SA_OK) return rc;
            den = mode.den;
        }
        const int n_chunks = (Nq + 63) / 64;
        const long n_tasks = BH * n_chunks;
        const long blocks = (n_tasks + 3) / 4;
        const dim3 grid((unsigned)blocks), block(256);
#define SA_QKV(DV_, ZO_) \
    qkv_kernel<DV_, ZO_><<<grid, block, 0, st>>>(q_codes, kv, out, H, Nq, W, n_chunks, n_tasks, scale, den, mode.eps)
        switch (dv) {
            case 32: if (mode.zero_one) SA_QKV(32, true); else SA_QKV(32, false); break;
            case 64: if (mode.zero_one) SA_QKV(64, true); else SA_QKV(64, false); break;
            default: if (mode.zero_one) SA_QKV(128, true); else SA_QKV(128, false); break;
        }
#undef SA_QKV
        int rc = sa::check_launch("sa_additive_attention(Q(K^T V))");
        if (rc == SA_OK && mode.xq)
            rc = sa_quantize_act_half(out, BH * Nq * dv, mode.act_inv_scale, mode.xq, mode.xh, stream);
        return rc;
    }
    return SA_OK;
}

size_t up256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

extern "C" int sa_additive_attention(const uint64_t *q_codes, const uint64_t *k_codes,
                                     const float *v, float *out, int B, int H, int Nq, int Nk,
                                     int nbits, int dv, float scale, float *kv, int phases,
                                     void *workspace, size_t workspace_bytes, void *stream) {
    sa::clear_error();
    return run_additive(q_codes, k_codes, v, out, B, H, Nq, Nk, nbits, dv, scale, kv, phases, workspace, workspace_bytes,
                        stream, AddMode{});
}

int sa::additive_attention_fused(const uint64_t *q_codes, const uint64_t *k_codes, const float *v, float *out, bool want_out,
                                 int B, int H, int N, int nbits, int dv, float scale, float *kv, int8_t *xq, _Float16 *xh,
                                 float act_inv_scale, void *workspace, size_t workspace_bytes, void *stream) {
    AddMode mode;
    mode.want_out = want_out;
    mode.xq = xq;
    mode.xh = xh;
    mode.act_inv_scale = act_inv_scale;
    return run_additive(q_codes, k_codes, v, out, B, H, N, N, nbits, dv, scale, kv, 3, workspace, workspace_bytes, stream, mode);
}

namespace {

// Workspace of sa_linear_attention_01: K^T V partials | their bit counts | normalisers [B*H, Nq] (vector-ALU phase 2).
struct ZeroOneLayout {
    size_t add, counts, den, total;
};

ZeroOneLayout zero_one_layout(int B, int H, int Nq, int Nk, int nbits, int dv) {
    ZeroOneLayout L;
    L.add = up256(sa_additive_attention_workspace_bytes(B, H, Nk, nbits, dv));
    L.counts = L.add;
    L.den = L.counts + up256(L.add / dv);         // one int32 per row of dv floats of the partials
    L.total = L.den + up256((size_t)B * H * (Nq > 0 ? Nq : 1) * sizeof(int32_t));
    return L;
}

}  // namespace

extern "C" size_t sa_linear_attention_01_workspace_bytes(int B, int H, int Nq, int Nk, int nbits, int dv) {
    if (B <= 0 || H <= 0 || Nq < 0 || Nk < 0 || nbits <= 0 || dv <= 0 || nbits % 64) return 0;
    return zero_one_layout(B, H, Nq, Nk, nbits, dv).total;
}

extern "C" int sa_linear_attention_01(const uint64_t *q_codes, const uint64_t *k_codes, const float *v, float *out,
                                      int B, int H, int Nq, int Nk, int nbits, int dv, float eps, float *kv,
                                      int32_t *ksum, int phases, void *workspace, size_t workspace_bytes,
                                      void *stream) {
    sa::clear_error();
    SA_REQUIRE(phases >= 1 && phases <= 7 && (phases & 3) != 0, SA_ERR_INVALID,
               "sa_linear_attention_01: phases must be 1, 2 or 3, optionally + 4");
    SA_REQUIRE(B >= 0 && H >= 0 && Nq >= 0 && Nk >= 0 && nbits > 0 && dv > 0, SA_ERR_INVALID,
               "sa_linear_attention_01: negative size");
    SA_REQUIRE(nbits % 64 == 0 && nbits <= 4096, SA_ERR_SHAPE,
               "sa_linear_attention_01: nbits %d must be a multiple of 64, at most 4096", nbits);
    SA_REQUIRE((long)Nk * nbits < (1L << 31), SA_ERR_SHAPE, "sa_linear_attention_01: the normaliser does not fit int32");
    SA_REQUIRE(eps > 0.0f && eps - eps == 0.0f, SA_ERR_INVALID, "sa_linear_attention_01: eps must be positive and finite");
    SA_REQUIRE((long)B * H < (1L << 20), SA_ERR_SHAPE, "sa_linear_attention_01: B*H too large");
    if ((long)B * H == 0) return SA_OK;
    SA_REQUIRE(ksum != nullptr, SA_ERR_INVALID, "sa_linear_attention_01: ksum is NULL");
    SA_REQUIRE(sa::aligned16(ksum) && sa::aligned16(workspace) && sa::aligned16(q_codes) && sa::aligned16(k_codes),
               SA_ERR_ALIGN, "sa_linear_attention_01: pointers must be 16-byte aligned");
    const size_t need = sa_linear_attention_01_workspace_bytes(B, H, Nq, Nk, nbits, dv);
    SA_REQUIRE(workspace != nullptr && workspace_bytes >= need, SA_ERR_WORKSPACE,
               "sa_linear_attention_01: workspace of %zu bytes needed, %zu given", need, workspace_bytes);
    if (phases & 2)
        SA_REQUIRE(Nq == 0 || (q_codes != nullptr && out != nullptr), SA_ERR_INVALID,
                   "sa_linear_attention_01: phase 2 needs q_codes and out");
    const ZeroOneLayout L = zero_one_layout(B, H, Nq, Nk, nbits, dv);
    uint8_t *ws = static_cast<uint8_t *>(workspace);
    AddMode mode;
    mode.zero_one = true;
    mode.ksum = ksum;
    mode.ksum_part = reinterpret_cast<int32_t *>(ws + L.counts);
    mode.den = reinterpret_cast<int32_t *>(ws + L.den);
    mode.eps = eps;
    return run_additive(q_codes, k_codes, v, out, B, H, Nq, Nk, nbits, dv, 1.0f, kv, phases, workspace, L.add, stream, mode);
}

extern "C" int sa_dwconv3x3(const float *v, const float *w, const float *bias_or_null, float *out, int accumulate,
                            int B, int gh, int gw, int E, void *stream) {
    sa::clear_error();
    SA_REQUIRE(B >= 0 && gh >= 0 && gw >= 0 && E >= 0, SA_ERR_INVALID, "sa_dwconv3x3: negative size");
    SA_REQUIRE(E % 4 == 0, SA_ERR_SHAPE, "sa_dwconv3x3: E (%d) must be a multiple of 4", E);
    const long n_tokens = (long)B * gh * gw;
    if (n_tokens == 0 || E == 0) return SA_OK;
    SA_REQUIRE(v && w && out, SA_ERR_INVALID, "sa_dwconv3x3: NULL buffer");
    SA_REQUIRE(v != out, SA_ERR_INVALID, "sa_dwconv3x3: out must not be v (neighbours are read after they would be written)");
    SA_REQUIRE(sa::aligned16(v) && sa::aligned16(w) && sa::aligned16(bias_or_null) && sa::aligned16(out), SA_ERR_ALIGN,
               "sa_dwconv3x3: pointers must be 16-byte aligned");
    // Outputs of a thread: four below each other (1.5 loads of a neighbour each instead of 3 and 9) once that still gives every SIMD
    // a wavefront; two where there are only two rows (64 x 2 x 98 x 768 30.3 -> 27.8 us, 8 x 2 x 8192 x 256 75 -> 65, where one
    // output each takes 38.8 and 107); of a single row four tokens beside each other (64 x 197 x 768 50.2 -> 15.8, 8 x 16384 x 256
    // 137 -> 41, one each 37 and 105).  From three rows on four (64 x 3 x 66 x 768 24.7, one each 49).
    const long n = n_tokens * (E / 4);
    const bool many = n >= 4L * 65536, line = many && gh == 1;
    if (line) std::swap(gh, gw);
    const int ry = !many ? 1 : gh == 2 && !line ? 2 : 4, strips = (gh + ry - 1) / ry;
    const long total = (long)B * strips * gw * (E / 4), blocks = (total + 255) / 256;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_dwconv3x3: too many elements");
    const sa::FastDiv by_e4((uint32_t)(E / 4)), by_gw((uint32_t)gw), by_strips((uint32_t)strips);
    const bool small = total < (1L << 31);
    auto go = [&](auto kernel) {
        kernel<<<dim3((unsigned)blocks), dim3(256), 0, sa::as_stream(stream)>>>(v, w, bias_or_null, out, accumulate, total, gh, gw, E / 4,
                                                                                strips, by_e4, by_gw, by_strips);
    };
    if (ry == 1) go(dwconv3x3_kernel<1, true, false>);
    else if (line) small ? go(dwconv3x3_kernel<4, true, true>) : go(dwconv3x3_kernel<4, false, true>);
    else if (ry == 2) small ? go(dwconv3x3_kernel<2, true, false>) : go(dwconv3x3_kernel<2, false, false>);
    else small ? go(dwconv3x3_kernel<4, true, false>) : go(dwconv3x3_kernel<4, false, false>);
    return sa::check_launch("sa_dwconv3x3");
}
