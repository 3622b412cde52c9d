// K^T V and Q (K^T V) of the additive attention (Eq. 3, O_Add; Sec. 4.1) on the matrix cores.
//
// An Add layer is a contraction with a +-1 operand: KV[bit, c] = sum_n s(n, bit) V[n, c] and
// out[n, c] = scale * sum_bit s(n, bit) KV[bit, c], s = +1 where the code bit is set, else -1.
// +-1 is exact in bf16, and an fp32 value is exactly the sum of three bf16 terms (each rounded to
// nearest from what the previous ones left), so v_mfma_f32_32x32x16_bf16 against the three term
// planes of the fp32 operand adds exactly the values the Add layer adds, in fp32: the same
// arithmetic as sign-select-and-accumulate on the vector ALU, at the matrix cores' rate (the
// plain-VALU rate is 39 T adds/s on this chip; the three-plane bf16 form runs ~20 times faster).
//
//   K^T V   : M = code bits (one 64-bit word = two 32-bit tiles per wavefront), N = dv columns,
//             K = tokens, 16 per MFMA.  Every wavefront loads the V rows and code words of its own steps
//             into a ring of its own in LDS and makes the three terms in registers.  Token ranges are split
//             over workgroups; partial sums meet in ascending order (no float atomics), in Q(K^T V) itself
//             when they are few.
//   Q(K^T V): M = tokens (TM 32-token tiles per wavefront), N = dv columns, K = code bits.
//             K^T V is staged once per workgroup, transposed into its three planes.
//
// The +-1 operand of both is made with two vector operations per pair of elements, from dwords that hold one bit of
// each element 16 positions apart: a shift brings the two bits to the sign positions of the two bf16 halves, an
// and-or drops the rest and adds the exponent of 1.0.  For Q(K^T V) the query's own code words are such dwords (bit i and
// bit i + 16 are neighbours in K, and K^T V is staged in that order: K may be permuted as long as both operands are);
// for K^T V the key codes are staged as dwords of 16 code bits of two consecutive tokens.
#include <type_traits>

#include "common.h"
#include "gemm_common.h"

namespace {

using sa::AddFused;
using sa::FastDiv;
using sa::kWave;

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

// (a, b) = sum of three bf16 term pairs, exactly: each term is the round-to-nearest bf16 of what the
// previous terms left.  t[p] holds term p of a in its lower and of b in its upper half (one
// v_cvt_pk_bf16_f32 per term pair).
__device__ inline void split3_pair(float a, float b, uint32_t (&t)[3]) {
    v2f r = {a, b};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        t[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, v2bf));
        if (p < 2) {
            r[0] -= __builtin_bit_cast(float, t[p] << 16);
            r[1] -= __builtin_bit_cast(float, t[p] & 0xFFFF0000u);
        }
    }
}

// Two bf16 operand elements from the bits at positions 15 - sh and 31 - sh of x: +1.0 (0x3F80) for a clear and -1.0 for
// a set bit, the negative of what the code stands for (the sums are negated where they leave); with ZO ({0,1} codes)
// 0.0 and 1.0.
template <bool ZO>
__device__ inline uint32_t code_pair(uint32_t x, int sh) {
    if (ZO) return ((x >> (15 - sh)) & 0x00010001u) * 0x3F80u;
    return ((x << sh) & 0x80008000u) | 0x3F803F80u;
}

// ------------------------------------------------------------------------------ K^T V ----
// Workgroup: one (b, h), up to four code words, up to 64 columns, one token range; eight wavefronts.  A wavefront has WB (1 or
// 2) words and every PH-th 16-token step, and holds that whole [64 WB bits, DVC columns] accumulator.  Its V rows and code
// words come in by direct global -> LDS loads into a ring of its own, RING steps deep (registers for that many are not
// there), so nothing is shared until the end and there is no barrier in the loop.  From the ring a lane reads its own MFMA
// operands, V[8 tokens][its columns] and its tokens' code words, splits V into the three terms in registers and makes the
// +-1 operand of a 32-bit tile with three vector operations per pair of tokens.
// (With four words two wavefronts split the same V: a SIMD issues a vector instruction of one wavefront in 5.2 cycles
// but of two in 2.6, and four of those fit in the shadow of an MFMA.)
// The kernel before this one staged V's planes through LDS for four wavefronts that shared them; its phases - load, split,
// multiply, with a barrier or two per 64 tokens - added up instead of overlapping.
// The wavefronts' accumulators meet in LDS in ascending order.
constexpr int kKtvWaves = 8;

template <int DVC, int WB, int RING, bool ZO>
struct KtvLds {
    static constexpr int SLOT = 16 * DVC * 4 + 256;              // a step in the ring: V rows, code words
    static constexpr int RING_BYTES = kKtvWaves * RING * SLOT, BYTES = RING_BYTES + (ZO ? kKtvWaves * WB * 64 * 4 : 0);
    static_assert(RING_BYTES >= kKtvWaves * 32 * DVC * 4, "the final sum reuses the ring");
};

// dst is not __restrict__: a kernel that goes on to Q(K^T V) reads the same memory through AddFused::kv_in.
// ksum (ZO): int32 [splits][BH][nbits], the number of tokens of the range whose code bit is set.
// split and rest: of block = rest * splits + split, rest = (bh * n_groups + group) * n_cols + column group.  (Quotients by numbers that the
// launch knows are multiplications: divisions, five of them one after the other, came before the first load.  32 x 3136 tokens' attention
// 20.74 -> 20.52 us, layer of 32 x 784 x 64 31.93 -> 31.70; both products of 1 x 3 heads x 197 x 64 bits in one launch 7.4 -> 6.7.)
template <int DVC, int WB, int PH, int RING, bool ZO>
__device__ __forceinline__ void ktv_block(const uint64_t *__restrict__ k_codes, const float *__restrict__ v, float *dst,
                                          int32_t *__restrict__ ksum, long BH, int H, FastDiv by_h, int Nk, int W, int DV,
                                          int tokens_per_block, int part, int rest, uint8_t *ring_s) {
    constexpr int JT = DVC / 32, TB = 2 * WB;                    // 32-column and 32-bit tiles
    constexpr int PAIRS = kKtvWaves / PH, GW = PAIRS * WB;       // shares of words, words of a workgroup
    constexpr int TILE = 32 * DVC;                               // floats of one 32-bit tile
    constexpr int V_BYTES = 16 * DVC * 4, SLOT = KtvLds<DVC, WB, RING, ZO>::SLOT;
    constexpr int LOADS = V_BYTES / 1024 + 1;                    // direct loads of a step
    float *red_s = reinterpret_cast<float *>(ring_s);
    int32_t *cnt_s = reinterpret_cast<int32_t *>(ring_s + KtvLds<DVC, WB, RING, ZO>::RING_BYTES);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int phase = wave / PAIRS;
    const int n_groups = (W + GW - 1) / GW, log_cols = __builtin_ctz((unsigned)DV / DVC);       // DV: 32, 64 or 128
    const int c0 = (rest & ((1 << log_cols) - 1)) * DVC, words = rest >> log_cols;
    const long bh = n_groups == 1 ? words : n_groups == 2 ? words >> 1 : words / n_groups;
    const int group = words - (int)bh * n_groups;
    const int b = (int)by_h((uint32_t)bh), h = (int)bh - b * H;
    const int w0 = group * GW + (wave % PAIRS) * WB;             // this wavefront's first word (may lie past the last one: idle)
    const int m = lane & 31, kg = lane >> 5;

    const int first = part * tokens_per_block;
    const int last = min(Nk, first + tokens_per_block);
    const int n_steps = w0 < W ? (last - first + 15) / 16 : 0;
    const size_t v_row = (size_t)H * DV * 4, c_row = (size_t)W * 8;                     // bytes
    const char *v_base = reinterpret_cast<const char *>(v + (((size_t)b * Nk + first) * H + h) * DV + c0);
    const char *c_base = reinterpret_cast<const char *>(k_codes + ((size_t)bh * Nk + first) * W + w0);

    // Step i into a slot of this wavefront's ring.  An address is the step's (the same in every lane) plus this lane's offset in
    // it; rows past the last token re-read the last one (step() blanks them), words past the last one likewise.
    uint8_t *ring = ring_s + wave * (RING * SLOT);
    const uint32_t ring_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)ring;
    constexpr int RPI = 1024 / (DVC * 4), LPR = DVC / 4;         // V rows per load, lanes per row
    const int c_tok = lane / (2 * WB) % 16, c_dw = min(lane % (2 * WB), 2 * (W - w0) - 1);     // (one word: the upper lanes repeat)
    // (32-bit lane offsets: at most RPI - 1 rows of H * DV floats, and with B * H < 2^20 heads that is 7 x 2^27 bytes with 32
    // columns to a workgroup, 3 x 2^29 with 64.  Whole rows beyond those go into the step's 64-bit part.)
    const uint32_t v_lane = (uint32_t)(lane / LPR) * (uint32_t)v_row + (lane % LPR) * 16;
    const uint32_t c_lane = (uint32_t)c_tok * (uint32_t)c_row + c_dw * 4;
    auto issue = [&](int i, int slot) {
        const char *vp = v_base + (size_t)i * 16 * v_row, *cp = c_base + (size_t)i * 16 * c_row;
        const int n = last - first - 16 * i;
        const uint32_t at = ring_base + slot * SLOT;
        if (n >= 16) {
#pragma unroll
            for (int k = 0; k < V_BYTES / 1024; ++k) sa::direct_load_16(vp + k * RPI * v_row, v_lane, at + k * 1024);
            sa::direct_load_4(cp, c_lane, at + V_BYTES);
        } else {
#pragma unroll
            for (int k = 0; k < V_BYTES / 1024; ++k) {
                const int row0 = min(k * RPI, n - 1);            // row min(k * RPI + lane / LPR, n - 1), in two parts
                sa::direct_load_16(vp + (size_t)row0 * v_row, (uint32_t)min(lane / LPR, n - 1 - row0) * (uint32_t)v_row + (lane % LPR) * 16,
                                   at + k * 1024);
            }
            sa::direct_load_4(cp, (uint32_t)min(c_tok, n - 1) * (uint32_t)c_row + c_dw * 4, at + V_BYTES);
        }
    };

    v16f acc[TB][JT];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int j = 0; j < JT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][j][r] = 0.0f;
    uint32_t cnt[TB] = {};                         // ZO: set bits among the even (lower half) and odd tokens of this lane
    int32_t total[TB] = {};
    const uint32_t pick = m < 16 ? 0x05040100u : 0x07060302u;    // the 16-bit half of a code dword that holds this lane's bit
    const int sh = 15 - (m & 15);

    // One step out of its slot: the +-1 operands, then column tile by column tile the three terms of V and their products.
    auto step = [&](int i, int slot) {
        const int n = last - first - 16 * i;
        const uint8_t *at = ring + slot * SLOT;
        float x[8][JT];
        uint32_t c[8][TB];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t *cw = reinterpret_cast<const uint32_t *>(at + V_BYTES) + (8 * kg + e) * TB;
            if constexpr (WB == 2) {
                const uint4 t = *reinterpret_cast<const uint4 *>(cw);
                c[e][0] = t.x; c[e][1] = t.y; c[e][2] = t.z; c[e][3] = t.w;
            } else {
                const uint2 t = *reinterpret_cast<const uint2 *>(cw);
                c[e][0] = t.x; c[e][1] = t.y;
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float *xp = reinterpret_cast<const float *>(at) + (8 * kg + e) * DVC + JT * m;
            if constexpr (JT == 2) {
                const float2 t = *reinterpret_cast<const float2 *>(xp);
                x[e][0] = t.x;
                x[e][1] = t.y;
            } else {
                x[e][0] = *xp;
            }
        }
        if (n < 16) {                                            // tokens that do not exist add nothing
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool in = 8 * kg + e < n;
#pragma unroll
                for (int j = 0; j < JT; ++j) x[e][j] = in ? x[e][j] : 0.0f;
                if (ZO) {
#pragma unroll
                    for (int q = 0; q < TB; ++q) c[e][q] = in ? c[e][q] : 0u;
                }
            }
        }
        v8bf sg[TB];
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            uint32_t d[4];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                const uint32_t pair = __builtin_amdgcn_perm(c[2 * e2 + 1][t], c[2 * e2][t], pick);
                d[e2] = code_pair<ZO>(pair, sh);
                if (ZO) cnt[t] += (pair >> (15 - sh)) & 0x00010001u;
            }
            sg[t] = __builtin_bit_cast(v8bf, make_uint4(d[0], d[1], d[2], d[3]));
        }
        sa::wait_lds_reads();                                    // this slot has been read ...
        if (i + RING * PH < n_steps) issue(i + RING * PH, slot);           // ... and is free for the step RING ahead
#pragma unroll
        for (int j = 0; j < JT; ++j) {
            uint32_t w[3][4];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                uint32_t t3[3];
                split3_pair(x[2 * e2][j], x[2 * e2 + 1][j], t3);
#pragma unroll
                for (int p = 0; p < 3; ++p) w[p][e2] = t3[p];
            }
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const v8bf vp = __builtin_bit_cast(v8bf, make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]));
#pragma unroll
                for (int t = 0; t < TB; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sg[t], vp, acc[t][j], 0, 0, 0);
            }
        }
    };

#pragma unroll
    for (int q = 0; q < RING; ++q)
        if (phase + q * PH < n_steps) issue(phase + q * PH, q);
    int slot = 0, done = 0;
    for (int i = phase; i < n_steps; i += PH) {
        const int later = (n_steps - 1 - i) / PH;                // steps of this wavefront after this one
        if (later >= RING - 1) sa::wait_loads_in_flight<(RING - 1) * LOADS>();
        else if (RING > 2 && later == 2) sa::wait_loads_in_flight<2 * LOADS>();
        else if (later == 1) sa::wait_loads_in_flight<LOADS>();
        else sa::wait_loads_in_flight<0>();
        step(i, slot);
        slot = slot + 1 == RING ? 0 : slot + 1;
        if (ZO && (++done & 0x1FFF) == 0) {        // before the 16-bit halves can overflow
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                total[t] += (int32_t)(cnt[t] & 0xFFFFu) + (int32_t)(cnt[t] >> 16);
                cnt[t] = 0;
            }
        }
    }
    __syncthreads();                               // every ring has been read

    // ---- the wavefronts' sums, in ascending order, one 32-bit tile of every share at a time; dst: [splits][BH][nbits][DV].  (Two words of
    //      more to a workgroup: in pairs of pairs.  They take the place of twice as many partials of half as many sums each, which one after
    //      the other they would be up to 7 % further from the exact sum than; so 3 % closer.)
    const bool in_pairs = PH == 8 && WB == 2 && n_groups > 1;
    //      With +-1 codes the operand was -1 for a set bit (the code bit as the sign bit), so the sum is negated here.
    const size_t row0 = (((size_t)part * BH + bh) * W + group * GW) * 64;
    const int rows_here = min(GW, W - group * GW) * 64;
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        if (t > 0) __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float *at = red_s + wave * TILE + (8 * (r >> 2) + 4 * kg + (r & 3)) * DVC + JT * m;
            if constexpr (JT == 2)
                *reinterpret_cast<float2 *>(at) = make_float2(acc[t][0][r], acc[t][1][r]);
            else
                *at = acc[t][0][r];
        }
        __syncthreads();
        for (int q = tid; q < PAIRS * TILE / 4; q += kKtvWaves * 64) {
            const int share = q / (TILE / 4);
            auto of = [&](int ph) { return reinterpret_cast<const f32x4 *>(red_s)[ph * PAIRS * (TILE / 4) + q]; };
            f32x4 a;
            if (in_pairs) {
                a = ((of(0) + of(1)) + (of(2) + of(3))) + ((of(PH / 2) + of(PH / 2 + 1)) + (of(PH / 2 + 2) + of(PH / 2 + 3)));
            } else {
                a = of(0);
#pragma unroll
                for (int ph = 1; ph < PH; ++ph) a += of(ph);
            }
            const int row = share * WB * 64 + t * 32 + q % (TILE / 4) / (DVC / 4), col = (q % (DVC / 4)) * 4;
            if (!ZO) a = -a;
            if (row < rows_here) *reinterpret_cast<f32x4 *>(dst + (row0 + row) * DV + c0 + col) = a;
        }
    }
    if (ZO && c0 == 0) {
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            int32_t n = total[t] + (int32_t)(cnt[t] & 0xFFFFu) + (int32_t)(cnt[t] >> 16);
            n += __shfl_xor(n, 32);
            if (kg == 0) cnt_s[wave * WB * 64 + t * 32 + m] = n;
        }
        __syncthreads();
        for (int q = tid; q < rows_here; q += kKtvWaves * 64) {
            int32_t n = cnt_s[q];
#pragma unroll
            for (int ph = 1; ph < PH; ++ph) n += cnt_s[ph * PAIRS * WB * 64 + q];
            ksum[row0 + q] = n;
        }
    }
}

template <int DVC, int WB, int PH, int RING, bool ZO>
__global__ __launch_bounds__(kKtvWaves * 64) void ktv_mfma_kernel(const uint64_t *__restrict__ k_codes, const float *__restrict__ v,
                                                                  float *__restrict__ dst, int32_t *__restrict__ ksum, long BH, int H,
                                                                  int Nk, int W, int DV, int splits, int tokens_per_block,
                                                                  FastDiv by_splits, FastDiv by_h) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[KtvLds<DVC, WB, RING, ZO>::BYTES];
    const int rest = (int)by_splits(blockIdx.x);
    ktv_block<DVC, WB, PH, RING, ZO>(k_codes, v, dst, ksum, BH, H, by_h, Nk, W, DV, tokens_per_block, (int)blockIdx.x - rest * splits, rest, lds);
}

// kv[i] = sum over splits of part[s][i].  G threads per 16 bytes: thread g takes a contiguous range of splits, s
// ascending, and the ranges meet in LDS in ascending order (with G = 1 the plain ascending sum).  With one thread per
// 16 bytes a small K^T V with many splits leaves the chip idle (64 KiB x 4 x 192 splits: 33 us on 64 workgroups).
template <int G, typename V4>
__device__ inline void reduce_splits(const V4 *__restrict__ part, V4 *__restrict__ dst, long n4, int splits, long i, int g, V4 *red) {
    V4 a = {};
    if (i < n4) {
        const int per = (splits + G - 1) / G, s0 = g * per, s1 = min(splits, s0 + per);
        int s = s0;
        for (; s + 4 <= s1; s += 4) {
            V4 p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) p[q] = part[(size_t)(s + q) * n4 + i];
#pragma unroll
            for (int q = 0; q < 4; ++q) a = (s + q == s0) ? p[q] : a + p[q];
        }
        for (; s < s1; ++s) a = (s == s0) ? part[(size_t)s * n4 + i] : a + part[(size_t)s * n4 + i];
    }
    if (G > 1) {
        red[threadIdx.x] = a;
        __syncthreads();
        if (g == 0 && i < n4) {
#pragma unroll
            for (int k = 1; k < G; ++k)
                if (k * ((splits + G - 1) / G) < splits) a = a + red[k * (256 / G) + threadIdx.x];
        }
    }
    if (g == 0 && i < n4) dst[i] = a;
}

// Workgroups below kv_blocks reduce K^T V, the rest (ksum_part not null) the bit counts.
template <int G>
__global__ __launch_bounds__(256) void ktv_sum_kernel(const f32x4 *__restrict__ part, f32x4 *__restrict__ kv, long n4, int splits,
                                                      unsigned kv_blocks, const i32x4 *__restrict__ ksum_part,
                                                      i32x4 *__restrict__ ksum, long k4) {
    __shared__ __attribute__((aligned(16))) f32x4 red[G > 1 ? 256 : 1];
    const int g = threadIdx.x / (256 / G), l = threadIdx.x % (256 / G);
    if (blockIdx.x < kv_blocks)
        reduce_splits<G>(part, kv, n4, splits, (long)blockIdx.x * (256 / G) + l, g, red);
    else
        reduce_splits<G>(ksum_part, ksum, k4, splits, (long)(blockIdx.x - kv_blocks) * (256 / G) + l, g,
                         reinterpret_cast<i32x4 *>(red));
}

// --------------------------------------------------------------------------- Q (K^T V) ----
// Workgroup: one (b, h), DVC (32 or 64) columns and a range of token tiles; NW wavefronts, TM 32-token tiles each per pass.
//
// K runs over the code bits in an order that makes the query's own code words the operand (see code_pair): step
// ks = 2 * half + s of a 32-bit half word, lane half kg, element e is bit 8 s + 4 kg + e / 2 + 16 (e % 2) of that half.

template <int DVC, int W, bool ZO>
struct QkvLds {
    static constexpr int STRIDE = W * 64 + 8;                    // bf16 elements per transposed K^T V row
    static constexpr int PLANE = DVC * STRIDE;                   // elements of a term plane
    // behind the planes: sums of the 16 subsets of every 4 bit counts (the normaliser), the counts
    static constexpr int BYTES = 3 * PLANE * 2 + (ZO ? W * 64 * 5 * 4 : 0);
};

// The codes of a wavefront's TM token tiles from tile0 on: this lane's query of each.
template <int W, int TM>
__device__ __forceinline__ void load_codes(const uint64_t *__restrict__ q_codes, long bh, int Nq, int tile0, uint64_t (&c)[TM][W]) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int n = min((tile0 + tm) * 32 + (int)(threadIdx.x & 31), Nq - 1);
        const uint64_t *cp = q_codes + ((size_t)bh * Nq + n) * W;
#pragma unroll
        for (int w = 0; w < W; ++w) c[tm][w] = cp[w];
    }
}

// Whether the codes of a wavefront's first tiles are asked for ahead of K^T V's planes, and those of the next ones while it multiplies
// these (32 x 3136 tokens x 1 head x 64 bits, both products 25.1 -> 24.7 us; {0,1} codes, Q(K^T V) of 8 x 4 x 16384 queries x 64 bits
// 29.9 -> 28.5, x 128 bits 37.4 -> 36.5).  Not {0,1} codes of 256 bits, for which 16 wavefronts do not leave the 16 registers: 22 of
// 128 were spilled on every tile's way (8 x 4 x 16384 queries 53.7 us at a tile's start, 64.8 ahead; 64 x 12 x 1100 queries 112 and
// 139).  Nor {0,1} codes where a wavefront has one tile: the tables of the normaliser come first (64 x 12 x 197 queries x 64 bits 16.3
// against 16.7 ahead), nor 256-bit codes there, whose registers cost a workgroup more (+-1, both products of 40 x 3 heads x 1024 tokens
// x 64 49.5 us, 51.5 ahead; 64 x 1 x 3136 56.5, 58.5).
template <int TM, int W, bool ZO>
constexpr bool kCodesAhead = ZO ? TM > 1 && W < 4 : TM > 1 || W < 4;

// SUMS: K^T V may come as partials.  AHEAD: the addresses of a tile's rows are made before the first one leaves.
// part and rest: of block = rest * blocks_per_bh + part, rest = bh * column groups + column group
template <int DVC, int W, int NW, int TM, bool ZO, bool SUMS, bool AHEAD>
__device__ __forceinline__ void qkv_block(const uint64_t *__restrict__ q_codes, const AddFused &f, int H, FastDiv by_h, int Nq, int DV,
                                          long BH, int tiles_per_block, int part, int rest, uint8_t *lds) {
    constexpr int JT = DVC / 32;
    constexpr int NBITS = W * 64;
    constexpr int STRIDE = QkvLds<DVC, W, ZO>::STRIDE, PLANE = QkvLds<DVC, W, ZO>::PLANE;
    uint16_t *kvt_s = reinterpret_cast<uint16_t *>(lds);
    int32_t *tab_s = reinterpret_cast<int32_t *>(lds + 3 * PLANE * 2), *ks_s = tab_s + NBITS * 4;

    const int tid = threadIdx.x, lane = tid & 63;
    constexpr int n_threads = NW * 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int log_cols = __builtin_ctz((unsigned)DV / DVC);           // DV: 32, 64 or 128
    const int c0 = (rest & ((1 << log_cols) - 1)) * DVC;
    const long bh = rest >> log_cols;
    const int b = (int)by_h((uint32_t)bh), h = (int)bh - b * H;
    const int m = lane & 31, kg = lane >> 5;
    uint64_t next[TM][W];                          // kCodesAhead: the codes of the tiles that come next
    if constexpr (kCodesAhead<TM, W, ZO>) load_codes<W, TM>(q_codes, bh, Nq, part * tiles_per_block + wave * TM, next);

    // K^T V -> the three planes: a task is the eight rows of one lane half of a step, one column
    constexpr int TASKS = (NBITS / 8 * DVC + n_threads - 1) / n_threads;
    auto bit_of = [&](int t, int e) {
        const int grp = t / DVC;                                   // (half * 2 + s) * 2 + kg
        return (grp >> 2) * 32 + ((grp >> 1) & 1) * 8 + (grp & 1) * 4 + (e >> 1) + 16 * (e & 1);
    };
    auto to_planes = [&](int t, const float (&x)[8]) {
        uint32_t w[3][4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            uint32_t t3[3];
            split3_pair(x[2 * e2], x[2 * e2 + 1], t3);
#pragma unroll
            for (int p = 0; p < 3; ++p) w[p][e2] = t3[p];
        }
#pragma unroll
        for (int p = 0; p < 3; ++p)
            *reinterpret_cast<uint4 *>(kvt_s + p * PLANE + t % DVC * STRIDE + t / DVC * 8) = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
    };
    // Two partials only where the launch has more than two workgroups for a CU: the sums' barriers cost a lone one more than the trip they save
    // (both products of 12 x 400 tokens x 64 10.55 us by quads, 10.44 below; 64 x 400 x 64 12.04, 11.93; 200 x 400 x 64 22.0, 22.6; 96 x 512 x 128
    // 19.6, 20.3).
    if (SUMS && W == 1 && f.splits > 1 && (f.splits > 2 || gridDim.x > 512)) {
        // Partials of 64-bit codes: summed on the way, in ascending order, and the first workgroup of the (b, h) leaves the sum in kv.
        // A thread sums four columns of a row, eight partials in flight: they come from other CUs, and one after the other each took
        // a trip of its own.  Both products of 32 x 3136 tokens x 1 head x 64 bits 17.1 -> 16.9 us, 4 x 12 x 3072 x 64 bits 29.1 -> 28.2,
        // 128 x 1 x 2000 x 64 35.6 -> 35.1; attention of the first with its hash 22.95 -> 22.65.
        constexpr int QUADS = NBITS * DVC / 4;
        static_assert(QUADS % n_threads == 0 && QUADS * 16 <= 3 * PLANE * 2, "sums where the planes go");
        f32x4 *sum_s = reinterpret_cast<f32x4 *>(lds);
#pragma unroll
        for (int i = 0; i < QUADS / n_threads; ++i) {
            const int t = tid + i * n_threads;
            const size_t at = ((size_t)bh * NBITS + t / (DVC / 4)) * DV + c0 + t % (DVC / 4) * 4, step = (size_t)BH * NBITS * DV;
            f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int s0 = 0; s0 < f.splits; s0 += 8) {
                f32x4 y[8];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (s0 + q < f.splits) y[q] = *reinterpret_cast<const f32x4 *>(f.kv_in + (s0 + q) * step + at);
                x = s0 == 0 ? y[0] : x + y[0];
#pragma unroll
                for (int q = 1; q < 8; ++q)
                    if (s0 + q < f.splits) x += y[q];
            }
            sum_s[t] = x;
            if (f.kv_out && part == 0) *reinterpret_cast<f32x4 *>(f.kv_out + at) = x;
        }
        __syncthreads();
        float x[TASKS][8];
#pragma unroll
        for (int i = 0; i < TASKS; ++i) {
            const int t = min(tid + i * n_threads, NBITS / 8 * DVC - 1);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[i][e] = reinterpret_cast<const float *>(lds)[bit_of(t, e) * DVC + t % DVC];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TASKS; ++i)
            if (tid + i * n_threads < NBITS / 8 * DVC) to_planes(tid + i * n_threads, x[i]);
    } else {
        for (int t = tid; t < NBITS / 8 * DVC; t += n_threads) {
            // Of 128 bits, and of two partials, one address and the others a constant away: made from bit_of each, both products of 400 x 20 tokens
            // x 32 x 128 bits took 8.10 us, so 7.95, of 24 x 7000 x 64 x 128 bits 42.3, 41.1.  Not for others (64 bits in one launch, layer of
            // 64 x 197 x 12 heads 196.4, 199.3; 256 bits 0.5 % longer over 200 sizes).
            constexpr bool NEAR = W == 2 || (W == 1 && SUMS);
            auto row = [&](int e) {
                return NEAR ? ((size_t)bh * NBITS + bit_of(t, 0)) * DV + c0 + t % DVC + ((e >> 1) + 16 * (e & 1)) * DV
                            : ((size_t)bh * NBITS + bit_of(t, e)) * DV + c0 + t % DVC;
            };
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = f.kv_in[row(e)];
            // Longer codes have fewer partials, of which the sums above have several quads a thread (4 x 8 heads x 4237 tokens x 128 bits 24.0,
            // there 24.2; 16 x 4 x 1600 21.0, 20.6; 8 x 8 x 1500 x 256 bits 27.1, 27.4).
            if constexpr (SUMS) {
                for (int s = 1; s < f.splits; ++s)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        x[e] += f.kv_in[NEAR ? (size_t)s * BH * NBITS * DV + row(e) : (((size_t)s * BH + bh) * NBITS + bit_of(t, e)) * DV + c0 + t % DVC];
                if (f.kv_out && part == 0)
#pragma unroll
                    for (int e = 0; e < 8; ++e) f.kv_out[row(e)] = x[e];
            }
            to_planes(t, x);
        }
    }
    if (ZO) {
        for (int j = tid; j < NBITS; j += n_threads) {
            int32_t c = f.ksum_in[(size_t)bh * NBITS + j];
            for (int s = 1; s < f.splits; s += 8) {
                int32_t y[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) y[q] = f.ksum_in[((size_t)min(s + q, f.splits - 1) * BH + bh) * NBITS + j];
#pragma unroll
                for (int q = 0; q < 8; ++q) c += s + q < f.splits ? y[q] : 0;
            }
            ks_s[j] = c;
            if (f.ksum_out && part == 0 && c0 == 0) f.ksum_out[(size_t)bh * NBITS + j] = c;
        }
        __syncthreads();
        for (int i = tid; i < NBITS * 4; i += n_threads) {
            const int32_t *k4 = ks_s + (i >> 4) * 4;
            tab_s[i] = ((i & 1) ? k4[0] : 0) + ((i & 2) ? k4[1] : 0) + ((i & 4) ? k4[2] : 0) + ((i & 8) ? k4[3] : 0);
        }
    }
    __syncthreads();

    const int n_tiles = (Nq + 31) / 32;
    const int tile_begin = part * tiles_per_block;
    const int tile_end = min(n_tiles, tile_begin + tiles_per_block);
    for (int tile0 = tile_begin + wave * TM; tile0 < tile_end; tile0 += NW * TM) {
        uint32_t code[TM][2 * W];
        float factor[TM];                         // ZO: 1 / (normaliser + eps) of this lane's query
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const uint64_t *here = q_codes + ((size_t)bh * Nq + min((tile0 + tm) * 32 + m, Nq - 1)) * W;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const uint64_t wd = kCodesAhead<TM, W, ZO> ? next[tm][w] : here[w];
                code[tm][2 * w] = (uint32_t)wd;
                code[tm][2 * w + 1] = (uint32_t)(wd >> 32);
            }
            if (ZO) {
                int32_t d = 0;
#pragma unroll
                for (int q = 0; q < 2 * W; ++q)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        d += tab_s[((q * 8 + 4 * kg + g) << 4) + ((code[tm][q] >> (16 * kg + 4 * g)) & 15u)];
                d += __shfl_xor(d, 32);
                factor[tm] = 1.0f / ((float)d + f.eps);
            }
#pragma unroll
            for (int q = 0; q < 2 * W; ++q) {     // the bits of lane half kg to where code_pair expects them
                code[tm][q] = ZO ? code[tm][q] >> (4 * kg) : code[tm][q] << (4 - 4 * kg);
            }
        }
        if (kCodesAhead<TM, W, ZO> && tile0 + NW * TM < tile_end) load_codes<W, TM>(q_codes, bh, Nq, tile0 + NW * TM, next);
        v16f acc[TM][JT];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int j = 0; j < JT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[tm][j][r] = 0.0f;

#pragma unroll
        for (int ks = 0; ks < NBITS / 16; ++ks) {
            v8bf a[TM];
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                uint32_t d[4];
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2)
                    d[e2] = code_pair<ZO>(code[tm][ks >> 1], (ZO ? 15 : 11) - 8 * (ks & 1) - e2);
                a[tm] = __builtin_bit_cast(v8bf, make_uint4(d[0], d[1], d[2], d[3]));
            }
#pragma unroll
            for (int j = 0; j < JT; ++j) {
                const int off = (j * 32 + m) * STRIDE + 16 * ks + 8 * kg;
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const v8bf kp = __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(kvt_s + p * PLANE + off));
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm) acc[tm][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[tm], kp, acc[tm][j], 0, 0, 0);
                }
            }
            // keep the steps apart: hoisting every operand read of the tile to the top costs hundreds of registers
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (tile0 + tm >= tile_end) continue;
            // a row's address is the tile's (the same in every lane) plus this lane's offset in it: no more than 4 rows of H * DV floats,
            // with B * H < 2^20 heads 2^31 bytes
            const size_t tile_at = (((size_t)b * Nq + (size_t)(tile0 + tm) * 32) * H + h) * DV + c0;
            int out_lane = lane;
            asm volatile("" : "+v"(out_lane));     // (made here: no registers for it beside the products)
            const int m = out_lane & 31, kg = out_lane >> 5;
            const uint32_t row_step = (uint32_t)H * DV, lane_at = (uint32_t)(4 * kg) * row_step + m;
            // FORMS: which of the three leave (1 fp32, 2 int8, 4 fp16; 8: AddFused::keep), or -1: asked for in every row.  Every wavefront of a launch runs this for
            // the first time, and few have more than one tile: what its instructions take to arrive counts.  So those of the common forms
            // have no others between them, and a row's address is made from the row's before, where it is used.  All made ahead of the tiles, as
            // the compiler does with tile_at + row * row_step, they were 300 instructions and most of the registers: Q(K^T V) of 32 x 3136
            // queries x 1 head x 64 bits 8.0 -> 6.6 us, both products of 1 x 3 x 197 x 64 bits 7.9 -> 7.4.  AHEAD: as AddFused::rows_ahead asks
            // (run_additive says when).
            auto store_rows = [&](auto whole_c, auto forms_c) {
                constexpr bool WHOLE = decltype(whole_c)::value;      // all 32 queries exist
                constexpr int FORMS = decltype(forms_c)::value;
                const bool keep = ZO && (FORMS < 0 ? f.keep : (FORMS & 8) != 0);
                const bool floats = FORMS < 0 ? f.out != nullptr : (FORMS & 1) != 0, bytes = FORMS < 0 ? f.xq != nullptr : (FORMS & 2) != 0,
                           halves = FORMS < 0 ? f.xh != nullptr : (FORMS & 4) != 0;
                size_t at = tile_at, ahead[16];
                auto next_row = [&](int r) {
                    if (r > 0) at += (size_t)(r % 4 ? 1 : 5) * row_step;
                    asm volatile("" : "+s"(at));
                };
                if constexpr (AHEAD) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        next_row(r);
                        ahead[r] = at;
                    }
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 8 * (r >> 2) + (r & 3);           // + 4 kg
                    if constexpr (AHEAD) at = ahead[r];
                    else next_row(r);
                    // (+-1: see code_pair.  __shfl, which allows for other widths, took 4 registers more than 256-bit codes leave.)
                    const float fr = ZO ? __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(16 * kg + 4 * row, __builtin_bit_cast(int, factor[tm])))
                                        : -f.scale;
                    if (WHOLE || (tile0 + tm) * 32 + row + 4 * kg < Nq) {
#pragma unroll
                        for (int j = 0; j < JT; ++j) {
                            const float val = fr * acc[tm][j][r];
                            if (floats) {
                                float *dst = reinterpret_cast<float *>(reinterpret_cast<char *>(f.out + at + j * 32) + lane_at * 4);
                                if (keep) *dst = val;
                                else __builtin_nontemporal_store(val, dst);
                            }
                            if (bytes) (f.xq + at + j * 32)[lane_at] = (int8_t)sa::requant_byte(val * f.act_inv_scale);
                            if (halves) *reinterpret_cast<_Float16 *>(reinterpret_cast<char *>(f.xh + at + j * 32) + lane_at * 2) = (_Float16)val;
                        }
                    }
                }
            };
            if (__builtin_expect((tile0 + tm) * 32 + 32 <= Nq, 1)) {
                if (ZO && f.keep) store_rows(std::true_type{}, std::integral_constant<int, ZO ? 9 : -1>{});
                else if (ZO || (!f.xq && !f.xh)) store_rows(std::true_type{}, std::integral_constant<int, 1>{});
                else if (!f.out && !f.xh) store_rows(std::true_type{}, std::integral_constant<int, 2>{});
                else if (!f.xh) store_rows(std::true_type{}, std::integral_constant<int, 3>{});
                else store_rows(std::true_type{}, std::integral_constant<int, -1>{});
            } else {
                store_rows(std::false_type{}, std::integral_constant<int, -1>{});
            }
        }
    }
}

template <int DVC, int W, int NW, int TM, bool ZO, bool AHEAD>
__global__ __launch_bounds__(NW * 64) void qkv_mfma_kernel(const uint64_t *__restrict__ q_codes, AddFused f, int H, int Nq, int DV,
                                                           long BH, int blocks_per_bh, int tiles_per_block, FastDiv by_blocks, FastDiv by_h) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[QkvLds<DVC, W, ZO>::BYTES];
    const int rest = (int)by_blocks(blockIdx.x);
    qkv_block<DVC, W, NW, TM, ZO, true, AHEAD>(q_codes, f, H, by_h, Nq, DV, BH, tiles_per_block, (int)blockIdx.x - rest * blocks_per_bh, rest, lds);
}

// ------------------------------------------------------------------- both, short sequences ----
// One workgroup does K^T V and Q(K^T V) of a (b, h) and DVC columns; what it reads of K^T V it wrote itself (splits = 1), so
// a barrier is all the order that takes.  Bound by latency for few sequences: 1 x 3 heads x 197 tokens x 64 bits 10.6 us in
// two launches, 7.5 in one; K^T V comes back from the caches it was just written to with many: 64 x 12 x 197 x 128 bits
// 33.2 -> 29.1, 64 x 3 x 197 x 64 bits 13.7 -> 9.9.  Kept in registers from the sums to the second product's planes, and the
// first queries' codes beside it, K^T V gained nothing for few sequences, and with many, which share a CU by twos at 128
// registers, it was slower (64 x 12 x 197 x 128 bits, 129 registers, 30.7 -> 39.1 us; x 64 bits 21.2 -> 22.4; 64 x 3 x 197 x 64
// 9.1 -> 10.0).
template <int DVC, int W, int PH, int WB, int RING>
__global__ __launch_bounds__(kKtvWaves * 64) void ktv_qkv_kernel(const uint64_t *__restrict__ k_codes, const float *__restrict__ v,
                                                                 float *kv, const uint64_t *__restrict__ q_codes, AddFused f,
                                                                 int H, int Nq, int Nk, int DV, long BH, FastDiv by_h) {
    constexpr int KB = KtvLds<DVC, WB, RING, false>::BYTES, QB = QkvLds<DVC, W, false>::BYTES;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[KB > QB ? KB : QB];
    static_assert(kKtvWaves / PH * WB == W, "a workgroup has all words");
    ktv_block<DVC, WB, PH, RING, false>(k_codes, v, kv, nullptr, BH, H, by_h, Nk, W, DV, (Nk + 15) & ~15, 0, blockIdx.x, lds);
    __syncthreads();
    qkv_block<DVC, W, kKtvWaves, 1, false, false, false>(q_codes, f, H, by_h, Nq, DV, BH, (Nq + 31) / 32, 0, blockIdx.x, lds);
}

// How the token tiles of a (b, h) are spread.
//  * Enough work to fill the chip with 32-tile passes: all columns up to 64 in one workgroup, 16 wavefronts with two tiles
//    each (a K^T V operand is then read once for both), one workgroup per CU and the tiles divided evenly: 50 us at 8 x 4
//    heads x 16384 queries x 256 bits x 64 columns (32 columns per workgroup: 57 us, the +-1 operand is made twice).
//  * Else 32 columns and eight tiles per workgroup: more, smaller workgroups (2 x 3 heads x 2000 x 128 bits x 128: 6.5 us
//    against 11; one DeiT-Tiny image: 5.0 against 5.4).
template <int W>
void launch_qkv_w(const uint64_t *q_codes, const AddFused &f, long BH, int H, int Nq, int dv, bool zo, hipStream_t st) {
    const int n_tiles = (Nq + 31) / 32;
#define SA_QKV_KERNEL(DVC_, NW_, TM_, ZO_, AHEAD_)                                                                                   \
    qkv_mfma_kernel<DVC_, W, NW_, TM_, ZO_, AHEAD_><<<grid, block, 0, st>>>(q_codes, f, H, Nq, dv, BH, per_bh, tiles_per_block, FastDiv(per_bh), FastDiv(H))
#define SA_QKV(DVC_, NW_, TM_)                                                                                                      \
    const dim3 grid((unsigned)(BH * (dv / DVC_) * per_bh)), block(NW_ * 64);                                                        \
    if (zo && f.rows_ahead) SA_QKV_KERNEL(DVC_, NW_, TM_, true, true);                                                              \
    else if (zo) SA_QKV_KERNEL(DVC_, NW_, TM_, true, false);                                                                        \
    else if (f.rows_ahead) SA_QKV_KERNEL(DVC_, NW_, TM_, false, true);                                                              \
    else SA_QKV_KERNEL(DVC_, NW_, TM_, false, false);
    if (dv >= 64 && BH * (dv / 64) * (n_tiles / 32) >= 256) {
        const long base = BH * (dv / 64);
        int per_bh = (int)((256 + base - 1) / base);
        const int tiles_per_block = (n_tiles + per_bh - 1) / per_bh;
        per_bh = (n_tiles + tiles_per_block - 1) / tiles_per_block;
        SA_QKV(64, 16, 2)
    } else {
        const int tiles_per_block = 8, per_bh = (n_tiles + 7) / 8;
        SA_QKV(32, 8, 1)
    }
#undef SA_QKV
#undef SA_QKV_KERNEL
}

}  // namespace

namespace sa {

// Tokens up to which one workgroup does both products of a (b, h): two rounds of its eight wavefronts' 32-token tiles.  Beyond
// that Q(K^T V) has tiles enough for several workgroups, which would each repeat or wait for K^T V.
constexpr int kShortTokens = 512;

// Shapes the matrix-core kernels take: K^T V any nbits (multiple of 64); Q(K^T V) 64-, 128- or 256-bit codes.
bool additive_mfma_ktv_supported(int nbits, int dv) { return nbits % 64 == 0 && (dv == 32 || dv == 64 || dv == 128); }

bool additive_mfma_qkv_supported(int nbits, int dv) {
    return (nbits == 64 || nbits == 128 || nbits == 256) && (dv == 32 || dv == 64 || dv == 128);
}

// Token splits of the K^T V pass: one workgroup per CU (every split writes a whole K^T V that has to be read again), and at
// least two steps for every wavefront.  quantum: tokens of one step of every wavefront.
static AdditiveMfmaPlan plan_splits(long heads, int groups, int quantum, int Nk) {
    AdditiveMfmaPlan p;
    p.groups = groups;
    const long base = heads * groups, units = ((long)Nk + 2 * quantum - 1) / (2 * quantum);
    long splits = (256 + base - 1) / base;
    if (splits > units) splits = units;
    if (splits < 1) splits = 1;
    if (splits > 256) splits = 256;
    const long per = ((long)Nk + splits - 1) / splits;
    p.tokens_per_block = (int)((per + 15) / 16 * 16);
    p.splits = (int)(((long)Nk + p.tokens_per_block - 1) / p.tokens_per_block);
    return p;
}

// Codes of more than two words: a workgroup has four of them (two wavefronts then take the same V), or two, which halves what the partials
// write and the sum reads and lets two workgroups read V.  Two where there are partials, unless V comes from memory (both products of 256
// bits, four words and two, us: 1 x 4 heads x 16384 tokens x 64 30.7, 27.8; 1 x 4 x 5471 23.4, 20.2; 2 x 4 x 8000 28.7, 26.4; 8 x 6 x 700 32.0, 29.2;
// 1 x 3 x 197 14.5, 13.5; V of 49 MB, 4 x 12 x 4000, 58.8, 59.9, but with no partials left, 16 x 12 x 1024, 62.8, 55.6; of 134 MB, 8 x 4 x 16384,
// 105.0, 107.5; without partials, 64 x 12 x 197, 56.0, 68.0), and not where Q(K^T V) would then sum them itself (32 x 1 x 3136 x 32 23.1, 24.2).
AdditiveMfmaPlan plan_additive_mfma(int B, int H, int Nk, int nbits, int dv) {
    const int W = nbits / 64;
    const long heads = (long)B * H * (dv > 64 ? dv / 64 : 1);
    if (W <= 2) return plan_splits(heads, 1, 16 * 8, Nk);
    const AdditiveMfmaPlan four = plan_splits(heads, (W + 3) / 4, 16 * 4, Nk), two = plan_splits(heads, (W + 1) / 2, 16 * 8, Nk);
    if (four.splits == 1 || (double)B * H * Nk * dv * 4 > (two.splits == 1 ? 64 : 32) * 1048576.0) return four;
    return two.splits == 1 || additive_mfma_sums_partials(two.splits, nbits, dv) == additive_mfma_sums_partials(four.splits, nbits, dv) ? two : four;
}

// Many short sequences: one word per wavefront and a short ring, so that two workgroups share a CU and one loads or sums while
// the other multiplies.  From the second round of workgroups on: 32 x 12 heads x 197 tokens x 128 bits 16.3 -> 11.9 us, 700
// tokens 28.2 -> 22.6, 1500 tokens 44.3 -> 39.4.  blocks: workgroups of up to 64 columns.
static bool ktv_many(long blocks) { return blocks > 256; }

int launch_ktv_mfma(const uint64_t *k_codes, const float *v, float *dst, int32_t *ksum, int B, int H, int Nk, int nbits, int dv,
                    const AdditiveMfmaPlan &p, bool zero_one, hipStream_t st) {
    const int W = nbits / 64;
    const long blocks = (long)B * H * p.groups * (dv > 64 ? dv / 64 : 1) * p.splits;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_additive_attention: grid too large");
    const dim3 grid((unsigned)blocks), block(kKtvWaves * 64);
    const bool many = ktv_many(blocks);
#define SA_KTV(DVC_, WB_, PH_, RING_)                                                                                          \
    if (zero_one) ktv_mfma_kernel<DVC_, WB_, PH_, RING_, true><<<grid, block, 0, st>>>(                                                 \
        k_codes, v, dst, ksum, (long)B * H, H, Nk, W, dv, p.splits, p.tokens_per_block, FastDiv(p.splits), FastDiv(H));                      \
    else ktv_mfma_kernel<DVC_, WB_, PH_, RING_, false><<<grid, block, 0, st>>>(                                                  \
        k_codes, v, dst, ksum, (long)B * H, H, Nk, W, dv, p.splits, p.tokens_per_block, FastDiv(p.splits), FastDiv(H));
#define SA_KTV_DV(DVC_)                       \
    if (W == 1 && many) { SA_KTV(DVC_, 1, 8, 2) }       \
    else if (W == 1) { SA_KTV(DVC_, 1, 8, 4) }          \
    else if (W == 2 && many) { SA_KTV(DVC_, 1, 4, 2) }  \
    else if (W == 2) { SA_KTV(DVC_, 2, 8, 4) }          \
    else if (p.groups == (W + 1) / 2) { SA_KTV(DVC_, 2, 8, 4) } \
    else { SA_KTV(DVC_, 2, 4, 4) }
    if (dv == 32) {
        SA_KTV_DV(32)
    } else {
        SA_KTV_DV(64)
    }
#undef SA_KTV_DV
#undef SA_KTV
    return check_launch("sa_additive_attention(K^T V)");
}

bool additive_mfma_one_launch(const AdditiveMfmaPlan &p, int Nq, int Nk, int nbits) {
    return p.splits == 1 && nbits <= 128 && Nq <= kShortTokens && Nk <= kShortTokens;
}

int launch_ktv_qkv(const uint64_t *k_codes, const float *v, float *kv, const uint64_t *q_codes, const AddFused &f, int B, int H,
                   int Nq, int Nk, int nbits, int dv, hipStream_t st) {
    const long BH = (long)B * H;
    // half of the columns per workgroup where that still leaves CUs idle
    const bool half = dv > 32 && BH * (dv / 32) <= 256;
    const int dvc = dv == 32 || half ? 32 : 64;
    const long blocks = BH * (dv / dvc);
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_additive_attention: grid too large");
    // The steps of a wavefront are those launch_ktv_mfma would give it, so that K^T V has the same bits either way.
    const bool many = ktv_many(BH * (dv > 64 ? dv / 64 : 1));
#define SA_BOTH(DVC_, W_, PH_, WB_, RING_)                                                                                      \
    ktv_qkv_kernel<DVC_, W_, PH_, WB_, RING_><<<dim3((unsigned)blocks), dim3(kKtvWaves * 64), 0, st>>>(k_codes, v, kv, q_codes, f, H, \
                                                                                                   Nq, Nk, dv, BH, FastDiv(H))
#define SA_BOTH_DV(DVC_)                                                                   \
    if (nbits == 64) { if (many) SA_BOTH(DVC_, 1, 8, 1, 2); else SA_BOTH(DVC_, 1, 8, 1, 4); } \
    else { if (many) SA_BOTH(DVC_, 2, 4, 1, 2); else SA_BOTH(DVC_, 2, 8, 2, 4); }
    if (dvc == 32) {
        SA_BOTH_DV(32)
    } else {
        SA_BOTH_DV(64)
    }
#undef SA_BOTH_DV
#undef SA_BOTH
    return check_launch("sa_additive_attention(K^T V, Q(K^T V))");
}

// K^T V partials that Q(K^T V) sums while it stages them: what a workgroup then reads stays within 128 KiB.
bool additive_mfma_sums_partials(int splits, int nbits, int dv) { return splits > 1 && (size_t)splits * nbits * dv * 4 <= 128 * 1024; }

int launch_ktv_sum(const float *part, float *kv, const int32_t *ksum_part, int32_t *ksum, long BH, int nbits, int dv, int splits,
                   hipStream_t st) {
    const long n4 = BH * nbits * dv / 4, k4 = ksum_part ? BH * nbits / 4 : 0;
    int G = 1;                                    // up to 16 threads per 16 bytes, until the chip has enough of them
    if (!additive_mfma_sums_partials(splits, nbits, dv))          // (the same plain sum whether or not Q(K^T V) takes it over)
        while (G < 16 && 4 * G <= splits && n4 * G < (1L << 17)) G *= 2;
    const long per = 256 / G;
    const long kv_blocks = (n4 + per - 1) / per, blocks = kv_blocks + (k4 + per - 1) / per;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_additive_attention: grid too large");
#define SA_SUM(G_)                                                                                                              \
    ktv_sum_kernel<G_><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(reinterpret_cast<const f32x4 *>(part),                     \
        reinterpret_cast<f32x4 *>(kv), n4, splits, (unsigned)kv_blocks, reinterpret_cast<const i32x4 *>(ksum_part),             \
        reinterpret_cast<i32x4 *>(ksum), k4)
    switch (G) {
        case 1: SA_SUM(1); break;
        case 2: SA_SUM(2); break;
        case 4: SA_SUM(4); break;
        case 8: SA_SUM(8); break;
        default: SA_SUM(16); break;
    }
#undef SA_SUM
    return check_launch("sa_additive_attention(sum of the partials)");
}

int launch_qkv_mfma(const uint64_t *q_codes, const AddFused &f, int B, int H, int Nq, int nbits, int dv, bool zero_one,
                    hipStream_t st) {
    const long BH = (long)B * H;
    switch (nbits) {
        case 64: launch_qkv_w<1>(q_codes, f, BH, H, Nq, dv, zero_one, st); break;
        case 128: launch_qkv_w<2>(q_codes, f, BH, H, Nq, dv, zero_one, st); break;
        case 256: launch_qkv_w<4>(q_codes, f, BH, H, Nq, dv, zero_one, st); break;
        default: return fail(SA_ERR_UNSUPPORTED, "sa_additive_attention: unsupported code width for the matrix-core path");
    }
    return check_launch("sa_additive_attention(Q(K^T V))");
}

}  // namespace sa
