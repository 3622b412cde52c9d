// LayerNorm, the Q, K, V projection and the hash of Q and K of a layer in one launch, for widths whose rows a workgroup can hold
// (E = 64 .. 256) and prepared weights:
//     (q, k, v)[row] = scale * Wqkv . codes(LayerNorm(x[row])),     bit j of q's code = [q[row, head] . proj[:, j] >= 0], k's alike
// Q and K leave as code words: 64 columns of them at a time go from the sums through LDS to the wavefronts that hash them, as in
// binarize_mfma.hip (three products of fp16 terms, a margin test, the defining chain for what that leaves open).  The chain's rows
// are the few with such bits, which are written out for it; V leaves as fp32.
//
// What it saves is a launch (its start, its prologue, the tail of the one before) and Q's and K's way to memory and back (4 E bytes a row
// each way for either: 67 MB at 16384 rows of E = 256).  What bounds it is a workgroup's own chain, with two wavefronts a SIMD: per
// chunk two barriers, the products of two planes, the fp16 split, three products a tile of the hash and the signs.  Hence the hash of a chunk
// runs one chunk behind its products, whose weights are in flight meanwhile (a ring of three units; stores behind the loads are not waited
// for).  Layers of 16384 rows, E = 256, four heads of 64, 256 bits: 112.7 us with two launches, 104.4 with one, of which prologue 4.4,
// LayerNorm 3.6, eight hashed chunks 2.55 each, V 2, chain 1.7 (in a trace: 42.4, norm_linear.hip and binarize_mfma.hip 21.1 + 20.9);
// 25088 rows of E = 64, two heads of 32, 64 bits: 39.1, 33.4 (in a trace 12.2, 8.7 + 7.7).  Fragments of the hash matrix in registers,
// with rows split once by the wavefront that has their sums, halve the LDS reads and make the chain longer: layers of 16384 rows 103.3
// where these are 98.0.
//
// With few rows (by_chunks) each workgroup makes one chunk: DeiT-Tiny layer of one image 41.5 -> 38.7 us, of which three launches were
// LayerNorm 2.9, projection 4.4, hash 6.6.
#include "common.h"
#include "gemm_common.h"
#include "gemm_mfma.h"
#include "hash_tile.h"
#include "layernorm.h"

namespace {

using namespace sa;

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8, kRows = 64, kChunk = 64;           // wavefronts 2 x 4 over rows x columns, rows, columns of a chunk

// NE: E / 64.  D: head width.  NB: code bits.  Of a chunk's rows (x heads, D = 32) a wavefront hashes 16 to NT tiles of 16
// columns.
template <int NE, int D, int NB>
struct NormHashShape {
    static constexpr int E = 64 * NE, S = D / 32;
    static constexpr int NT = D == 32 ? 4 : NB / 32, COLS = 16 * NT, GROUPS = NB / COLS;
    static constexpr int HEADS = kChunk / D;                 // of a chunk
    static_assert(HEADS * kRows / 16 * GROUPS == kWaves && (D == 64 || NB == 64), "a chunk's rows and columns, once");
    static constexpr int UNIT = kChunk * E, RING = 3;        // 64 rows of a plane of Wqkv
    static constexpr int TOTAL = UNIT / 1024, LOADS = (TOTAL + kWaves - 1) / kWaves;       // KiB of a unit, of a wavefront
    static constexpr int LIST = 96;                          // open bits of a wavefront
    static constexpr int TPC = kWaves * 64 / NB < 4 * S ? kWaves * 64 / NB : 4 * S, TASKS = 4 * S / TPC;      // threads of a hash column
    // LDS: ring, two chunks of staged rows (before them the codes of the normalised ones), fragments of the hash matrix, lists, masks, norms
    static constexpr int STAGE = RING * UNIT, STAGE_BYTES = kRows * kChunk * 4, FRAGS = STAGE + 2 * STAGE_BYTES, LISTS = FRAGS + NB * D * 4;
    static constexpr int MASKS = LISTS + kWaves * LIST * 8, NORMS = MASKS + 2 * NB / 8, COUNTS = NORMS + TPC * NB * 4, LDS_BYTES = COUNTS + kWaves * 4;
    static constexpr int PER_CU = D == 32 && NE == 1 ? 2 : 1;      // workgroups (what the registers allow)
    static_assert(kRows * E <= STAGE_BYTES && PER_CU * LDS_BYTES <= 160 * 1024, "LDS of a CU");
};

struct HashOut {
    const float *proj;                   // [D, NB]
    float *q, *k;                        // [T, E]: rows with open bits
    Tensors of;                          // the same, and where their codes go
    RowMap map;
};

// Sum over lanes l, l + 16, l + 32 and l + 48; all of them get it.
__device__ inline float sum_of_rows(float v) {
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const uint32_t r0 = r[0], r1 = r[1], s = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1));
    const auto t = __builtin_amdgcn_permlane16_swap(s, s, false, false);
    const uint32_t t0 = t[0], t1 = t[1];
    return __builtin_bit_cast(float, t0) + __builtin_bit_cast(float, t1);
}

// SPLIT: workgroup 3 NE r + c makes chunk c of its rows alone.
template <int NE, int D, int NB, bool SPLIT>
__global__ __launch_bounds__(kWaves * 64, D == 32 && NE == 1 ? 4 : 2) void norm_hash_kernel(NormRows norm, long n_rows, const int8_t *__restrict__ w,
                                                                                 float scale, HashOut h, float *__restrict__ v) {
    using S = NormHashShape<NE, D, NB>;
    constexpr int E = S::E, NT = S::NT, KS = S::S;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[S::LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 2, wc = wave & 3, fr = lane & 15, fg = lane >> 4;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    uint64_t *list = reinterpret_cast<uint64_t *>(lds + S::LISTS) + wave * S::LIST;
    int cnt = 0;                                             // entries of it (wave-uniform)

    // unit u: plane u % 2 of columns 64 (u / 2) ..
    auto issue = [&](int u, int slot) {
        const int8_t *base = w + (size_t)(u & 1) * 3 * E * E + (size_t)(u >> 1) * S::UNIT;
#pragma unroll
        for (int j = 0; j < S::LOADS; ++j) {
            const int kib = (j * kWaves + wave) % S::TOTAL;              // (past the end: the same bytes once more)
            const int c = kib * 64 + lane, r = c / (4 * NE);
            direct_load_16(base, (uint32_t)(r * E + swizzle_row<NE>(r, c % (4 * NE)) * 16), lds_base + slot * S::UNIT + kib * 1024);
        }
    };
    constexpr int UNITS = 6 * NE;
    const int only = SPLIT ? (int)(blockIdx.x % (3 * NE)) : 0;           // the chunk of a SPLIT workgroup
    const bool hashes = !SPLIT || only < 2 * NE;
    // this wavefront's rows to normalise, LPR lanes each
    constexpr int LPR = NE == 1 ? 16 : NE == 2 ? 32 : 64, LANES = 64 / LPR, STEPS = kRows / kWaves / LANES;
    const int l = lane % LPR, row0 = wave * (kRows / kWaves) + lane / LPR;
    const bool in = 4 * l < E;
    const int col = min(4 * l, E - 4);                                   // (lanes past the row: its end, not used; see row_or_zero)
    float4 xr[STEPS];
    auto load_rows = [&](long m0) {
#pragma unroll
        for (int i = 0; i < STEPS; ++i)
            xr[i] = *reinterpret_cast<const float4 *>(norm.x + (size_t)min(m0 + row0 + LANES * i, n_rows - 1) * E + col);
    };
    long m0 = (long)(SPLIT ? blockIdx.x / (3 * NE) : blockIdx.x) * kRows;
    if (m0 >= n_rows) return;
    if (blockIdx.x == 0) zero_words(norm.zero);
    load_rows(m0);
    const float4 gamma = *reinterpret_cast<const float4 *>(norm.gamma + col);
    const float4 beta = *reinterpret_cast<const float4 *>(norm.beta + col);

    // ---- the hash matrix, as fragments of its normalised columns (upper and lower fp16 terms).  Lane group q of a product's result
    //      has columns COLS / 4 q .. of a wavefront's COLS.
    const int hc = tid % NB, part = tid / NB;
    const bool mine = hashes && part < S::TPC;
    float hv[S::TASKS][8];
    auto k_of = [&](int i, int e) {
        const int j = part + i * S::TPC;                                 // task j: 32 (j / 4) + 4 (j % 4) and 16 further on
        return 32 * (j >> 2) + 16 * (e / 4) + 4 * (j & 3) + e % 4;
    };
    if (mine) {
#pragma unroll
        for (int i = 0; i < S::TASKS; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) hv[i][e] = h.proj[(size_t)k_of(i, e) * NB + hc];
    }
    issue(2 * only, 0);
    issue(2 * only + 1, 1);
    float *norms = reinterpret_cast<float *>(lds + S::NORMS);
    uint4 *frags = reinterpret_cast<uint4 *>(lds + S::FRAGS);
    uint64_t *zero_columns = reinterpret_cast<uint64_t *>(lds + S::MASKS), *unbounded_columns = zero_columns + NB / 64;      // bit: a column
    if (mine) {
        float n2 = 0.0f;                                                 // this thread's share of the norm
#pragma unroll
        for (int i = 0; i < S::TASKS; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) n2 = __builtin_fmaf(hv[i][e], hv[i][e], n2);
        norms[part * NB + hc] = column_norm(n2, hv);
    }
    __syncthreads();
    if (mine) {
        float n2 = 0.0f;
#pragma unroll
        for (int p = 0; p < S::TPC; ++p) n2 += norms[p * NB + hc];
        const uint64_t zero = __ballot(n2 == 0.0f), unbounded = __ballot(!(n2 < __builtin_inff()));
        if (part == 0 && lane == 0) {
            zero_columns[hc / 64] = zero;
            unbounded_columns[hc / 64] = unbounded;
        }
        // a column of no use (see binarize_mfma.hip) is left to the chain, unless it is all zeros
        const float inv = n2 >= kColumnMin2 && n2 < __builtin_inff() ? 1.0f / __builtin_sqrtf(n2) : 0.0f;
        const int c = hc % S::COLS, q = c / (S::COLS / 4), b = c % (S::COLS / 4), t = b / 4, rho = 4 * q + b % 4;
#pragma unroll
        for (int i = 0; i < S::TASKS; ++i) {
            const int j = part + i * S::TPC;
            uint32_t up[4], lo[4];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                float x[2];
#pragma unroll
                for (int o = 0; o < 2; ++o) x[o] = inv > 0.0f ? hv[i][2 * e2 + o] * inv * kColumnScale : 0.0f;
                split_f16_pair(x[0], x[1], up[e2], lo[e2]);
            }
            uint4 *at = frags + (((hc / S::COLS * NT + t) * KS + (j >> 2)) * 2) * 64 + (j & 3) * 16 + rho;
            at[0] = make_uint4(up[0], up[1], up[2], up[3]);
            at[64] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        }
    }

    auto staged = [&](int c, int r, int q) {
        return reinterpret_cast<v4f *>(lds + S::STAGE + (c & 1) * S::STAGE_BYTES + r * (kChunk * 4) + (q ^ (r & 15)) * 16);
    };
    auto work_off = [&]() {
        // A SPLIT workgroup's rows are staged still: nothing of them goes through memory, and the chain runs while the words are on their
        // way (layers of 197 x 192 37.1 -> 36.8 us, 1500 x 192 46.6 -> 45.9, 1000 x 256 of 256 bits 56.9 -> 56.0).
        if constexpr (SPLIT) {
#pragma unroll 1
            for (int t0 = 0; t0 < cnt; t0 += 64)
                if (t0 + lane < cnt) {
                    const uint64_t e = list[t0 + lane];
                    const uint32_t row = (uint32_t)e, t = row / (E / D);
                    const int col = (int)((e >> 32) & 0xffffu), q0 = (int)(row % (E / D) % S::HEADS) * (D / 4);
                    float cols[D], acc = 0.0f;
#pragma unroll
                    for (int k = 0; k < D; ++k) cols[k] = h.proj[(size_t)k * NB + col];
#pragma unroll
                    for (int q = 0; q < D / 4; ++q) {
                        const v4f x = *staged(only, (int)((long)t - m0), q0 + q);
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc = __builtin_fmaf(x[i], cols[4 * q + i], acc);
                    }
                    wait_loads_in_flight<0>();               // the word this bit lives in has been stored
                    if ((acc >= 0.0f) != (bool)((e >> 48) & 1u))
                        atomicXor(reinterpret_cast<unsigned long long *>((((e >> 49) & 1u) ? h.of.codes1 : h.of.codes0) + h.map.row_words(row) + (col >> 6)),
                                  1ull << (col & 63));
                }
        } else {
            wait_loads_in_flight<0>();                       // the words these bits live in and the rows have been stored
#pragma unroll 1
            for (int t0 = 0; t0 < cnt; t0 += 64)
                if (t0 + lane < cnt) settle_entry<D, 16>(list[t0 + lane], h.of, h.proj, NB, 0, h.map);
        }
        cnt = 0;
    };

    // what this wavefront hashes of a chunk
    const int group = S::GROUPS == 1 ? 0 : wave % S::GROUPS;
    const int head = S::HEADS == 2 ? wave & 1 : 0;
    const int row16 = wave / (S::GROUPS * S::HEADS) * 16;                // first of its rows
    uint32_t zeros = 0;                                                  // which of this lane's columns are all zeros (the barrier comes below)

    const int units = SPLIT ? 2 * only + 2 : UNITS;
    int slot = 0, ahead = 2 * only + 2;                      // the unit's place in the ring; the next unit to load
    // Stores that this wavefront issued at the end of the last chunk, at least: behind the loads that either half of the next one waits
    // for, which need not wait for them as well.
    int stores = 0;
    for (;;) {
        const long next_m0 = m0 + (long)gridDim.x * kRows;
        const bool more = !SPLIT && next_m0 < n_rows;
        // ---- LayerNorm: codes to LDS, from there to all wavefronts as operands
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const float4 x[1] = {row_or_zero(xr[i], in)};
            float mean, rstd, y[4];
            row_stats<LPR, 1>(x, l, E, norm.eps, mean, rstd);
            normalise(x[0], mean, rstd, gamma, beta, y);
            const int r = row0 + LANES * i;
            if (in) *reinterpret_cast<uint32_t *>(lds + S::STAGE + r * E + swizzle_row<NE>(r, l / 4) * 16 + l % 4 * 4) = codes_of(y, norm.inv_scale);
        }
        __syncthreads();
        if (hashes) {
            const int bit0 = S::COLS * group + 4 * NT * fg;
            zeros = (uint32_t)(zero_columns[bit0 / 64] >> bit0 % 64);
        }
        uint4 xf[2][NE];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int s = 0; s < NE; ++s) {
                const int r = wr * 32 + 16 * i + fr;
                xf[i][s] = *reinterpret_cast<const uint4 *>(lds + S::STAGE + r * E + swizzle_row<NE>(r, 4 * s + fg) * 16);
            }

        // where the code words of this wavefront's rows lie: word_at + head * N words
        size_t word_at;
        {
            const uint32_t t = (uint32_t)min(m0 + row16 + fr, n_rows - 1), b = h.map.by_n(t), n = t - b * (uint32_t)h.map.N;
            word_at = (size_t)b * h.map.H * h.map.N + n;
        }
        // ---- chunk c of the projection.  Products are computed transposed (weights down, rows across): a lane holds four consecutive
        //      columns of rows 32 wr + lane % 16 and 16 further on.
        v4i acc[2];
        auto multiply = [&](int p) {
            // this unit is there, the next one need not be; everyone is through with the one before, whose place the unit after
            // the next one takes
            if (!(ahead <= units || more)) wait_loads_in_flight<0>();
            else if (stores == 0) wait_loads_in_flight<S::LOADS>();
            else if (stores == 1) wait_loads_in_flight<S::LOADS + 1>();
            else wait_loads_in_flight<S::LOADS + 2>();
            __syncthreads();
            const int to = slot == 0 ? 2 : slot - 1;
            if (ahead < units) issue(ahead, to);
            else if (more) issue(ahead - UNITS, to);
            ++ahead;
#pragma unroll
            for (int s = 0; s < NE; ++s) {
                const int r = wc * 16 + fr;
                const uint4 b = *reinterpret_cast<const uint4 *>(lds + slot * S::UNIT + r * E + swizzle_row<NE>(r, 4 * s + fg) * 16);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, b), __builtin_bit_cast(v4i, xf[i][s]),
                                                                   p == 0 && s == 0 ? v4i{0, 0, 0, 0} : acc[i], 0, 0, 0);
            }
            slot = slot == 2 ? 0 : slot + 1;
        };
        // A chunk's sums are Q's or K's (staged) or V's; between the two halves of its products come the operands of the chunk before,
        // behind them that one's hash.  A chunk of staged rows is read behind a barrier and written over behind another.
        // (A SPLIT workgroup's only chunk is hashed with no products beside it.)
        auto chunk = [&](int c, auto hash_c, auto staged_c) {
            constexpr bool HASH = decltype(hash_c)::value, STAGED = decltype(staged_c)::value, PRODUCTS = !(SPLIT && HASH);
            // (the lane's addresses are made here, not kept from chunk to chunk: the registers are needed)
            int of_lane = lane;
            asm volatile("" : "+v"(of_lane));
            const int fr = of_lane & 15, fg = of_lane >> 4;
            // row row16 + fr of the chunk's head, this lane's k = 32 s + 16 o + 4 fg ..
            v4f x[KS][2];
            if constexpr (PRODUCTS) multiply(0);
            else __syncthreads();
            if constexpr (HASH) {
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int o = 0; o < 2; ++o) x[s][o] = *staged(c - 1, row16 + fr, head * (D / 4) + 8 * s + 4 * o + fg);
            }
            if constexpr (PRODUCTS) multiply(1);
            if constexpr (HASH) {
                const bool second = c - 1 >= NE;
                const int head0 = (second ? c - 1 - NE : c - 1) * S::HEADS + head;       // of the layer
                constexpr int PAIRS = KS * NT / 2;           // of tiles, step by step
                uint4 fr2[2][2][2];                          // [pair's parity][tile][upper, lower]
                auto read_pair = [&](int pair) {
                    const int s = pair / (NT / 2), t = pair % (NT / 2) * 2;
#pragma unroll
                    for (int o = 0; o < 2; ++o)
#pragma unroll
                        for (int term = 0; term < 2; ++term) fr2[pair & 1][o][term] = frags[(((group * NT + t + o) * KS + s) * 2 + term) * 64 + of_lane];
                };
                read_pair(0);
                v8h xh[KS], xl[KS];
                float nx2 = 0.0f;
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int o = 0; o < 2; ++o)
#pragma unroll
                        for (int e = 0; e < 4; ++e) nx2 = __builtin_fmaf(x[s][o][e], x[s][o][e], nx2);
                nx2 = sum_of_rows(nx2);
                auto split = [&](float unit) {
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        uint32_t up[4], lo[4];
#pragma unroll
                        for (int o = 0; o < 2; ++o) {
                            const v4f y = x[s][o] * unit;
                            split_f16_pair(y[0], y[1], up[2 * o], lo[2 * o]);
                            split_f16_pair(y[2], y[3], up[2 * o + 1], lo[2 * o + 1]);
                        }
                        xh[s] = __builtin_bit_cast(v8h, make_uint4(up[0], up[1], up[2], up[3]));
                        xl[s] = __builtin_bit_cast(v8h, make_uint4(lo[0], lo[1], lo[2], lo[3]));
                    }
                };
                // rows of ordinary magnitude split as they are, others are brought to |x| ~ 1 first (hash_margin.h)
                float unit = 1.0f;
                bool zero = false;                           // a row of zeros: hash_tile.h
                if (__ballot(!(nx2 >= kOrdinaryMin2 && nx2 <= kOrdinaryMax2)) != 0) {        // wave-uniform
                    int e = 0;
                    if (nx2 > 0.0f && nx2 < __builtin_inff()) e = __builtin_amdgcn_frexp_expf(nx2) / 2;
                    unit = __builtin_amdgcn_ldexpf(1.0f, -e);
                    split(unit);
                    zero = nx2 == 0.0f && scale_is_exact(scale);
#pragma unroll
                    for (int q = 0; q < NB / 64; ++q) zero = zero && unbounded_columns[q] == 0;
                } else {
                    split(1.0f);
                }
                float keep = nx2 < __builtin_inff() ? __builtin_fmaxf(hash_theta(D) * __builtin_sqrtf(nx2), kKeepFloor) * unit * kColumnScale
                                                  : __builtin_inff();
                if (zero) keep = -1.0f;
                // Two tiles' products by turns, their fragments read a pair ahead (the first pair's before the rows are split): left to
                // itself the compiler read most of them a product ahead (layer of 16384 x 256, 256 bits 100.8 -> 99.6 us).
                v4f z[NT];
#pragma unroll
                for (int pair = 0; pair < PAIRS; ++pair) {
                    if (pair + 1 < PAIRS) read_pair(pair + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int part = 0; part < 3; ++part)             // xh rh, xh rl, xl rh
#pragma unroll
                        for (int o = 0; o < 2; ++o) {
                            const int s = pair / (NT / 2), t = pair % (NT / 2) * 2 + o;
                            z[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, fr2[pair & 1][o][part == 1]), part == 2 ? xl[s] : xh[s],
                                                                          s == 0 && part == 0 ? v4f{0.0f, 0.0f, 0.0f, 0.0f} : z[t], 0, 0, 0);
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
                uint32_t neg = 0;                            // bit q: sign of element q (-0 is open anyway)
                float smallest = __builtin_inff();
#pragma unroll
                for (int q = 4 * NT - 1; q >= 0; --q) {
                    const float zq = z[q / 4][q % 4];
                    neg = __builtin_amdgcn_alignbit(neg, __builtin_bit_cast(uint32_t, zq), 31);
                    smallest = __builtin_fminf(smallest, __builtin_fabsf(zq));
                }
                const uint32_t bits = ~neg & (uint32_t)((1ull << (4 * NT)) - 1);
                const long m = m0 + row16 + fr;
                const int bit0 = S::COLS * group + 4 * NT * fg;          // this lane's first column
                uint8_t *dst = reinterpret_cast<uint8_t *>((second ? h.of.codes1 : h.of.codes0) + (word_at + (size_t)head0 * h.map.N) * (NB / 64)) + bit0 / 8;
                if (m < n_rows) {
                    if constexpr (NT == 8) *reinterpret_cast<uint32_t *>(dst) = bits;
                    else if constexpr (NT == 4) *reinterpret_cast<uint16_t *>(dst) = (uint16_t)bits;
                    else *dst = (uint8_t)bits;
                }
                if (__ballot(m < n_rows && !(smallest > keep)) != 0) {   // wave-uniform
                    uint32_t open = 0;
#pragma unroll
                    for (int q = 0; q < 4 * NT; ++q) open |= (uint32_t)(!(__builtin_fabsf(z[q / 4][q % 4]) > keep)) << q;
                    if (m >= n_rows) open = 0;
                    if (keep < __builtin_inff()) open &= ~zeros;
                    // rows with open bits go out for the chain: all four lanes of such a row have a quarter of it
                    const uint64_t any = __ballot(open != 0);
                    if (!SPLIT && ((any >> fr | any >> (fr + 16) | any >> (fr + 32) | any >> (fr + 48)) & 1u)) {
                        float *to = (second ? h.k : h.q) + (size_t)m * E + head0 * D + 4 * fg;
#pragma unroll
                        for (int s = 0; s < KS; ++s)
#pragma unroll
                            for (int o = 0; o < 2; ++o) *reinterpret_cast<v4f *>(to + 32 * s + 16 * o) = x[s][o];
                    }
                    while (__ballot(open != 0) != 0) {       // wave-uniform
                        if (cnt + 64 > S::LIST) work_off();
                        const uint64_t pm = __ballot(open != 0);
                        if (open) {
                            const int pos = __builtin_ctz(open);
                            const int at = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(pm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pm, 0u));
                            list[at] = open_bit((uint32_t)m * (E / D) + head0, bit0 + pos, (bits >> pos) & 1u, second);
                            open &= open - 1u;
                        }
                        cnt += __builtin_popcountll(pm);
                    }
                }
            }
            if constexpr (!PRODUCTS) return;
            stores = HASH && m0 + row16 < n_rows ? 1 : 0;
            if constexpr (!STAGED) stores = (m0 + wr * 32 < n_rows) + (m0 + wr * 32 + 16 < n_rows);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = wr * 32 + 16 * i + fr;
                const v4f y = {__builtin_fmaf((float)acc[i][0], scale, 0.0f), __builtin_fmaf((float)acc[i][1], scale, 0.0f),
                               __builtin_fmaf((float)acc[i][2], scale, 0.0f), __builtin_fmaf((float)acc[i][3], scale, 0.0f)};
                if constexpr (STAGED) *staged(c, r, wc * 4 + fg) = y;
                else if (m0 + r < n_rows) *reinterpret_cast<v4f *>(v + (size_t)(m0 + r) * E + (c - 2 * NE) * kChunk + wc * 16 + 4 * fg) = y;
            }
        };
        if constexpr (SPLIT) {
            if (!hashes) return chunk(only, std::false_type{}, std::false_type{});
            chunk(only, std::false_type{}, std::true_type{});
            chunk(only + 1, std::true_type{}, std::false_type{});
            return work_off();
        }
        chunk(0, std::false_type{}, std::true_type{});
#pragma unroll 1
        for (int c = 1; c < 2 * NE; ++c) chunk(c, std::true_type{}, std::true_type{});
        chunk(2 * NE, std::true_type{}, std::false_type{});
        if (more) load_rows(next_m0);
#pragma unroll 1
        for (int c = 2 * NE + 1; c < 3 * NE; ++c) chunk(c, std::false_type{}, std::false_type{});
        if (!more) break;
        m0 = next_m0;
        ahead -= UNITS;
        __syncthreads();                                     // the staged rows have been read: the codes' place is free
    }

    // what is left open, pooled: 64 entries a pass, passes side by side on the wavefronts
    wait_loads_in_flight<0>();                               // this wavefront's words and rows have been stored
    int *counts = reinterpret_cast<int *>(lds + S::COUNTS);
    if (lane == 0) counts[wave] = cnt;
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) total += counts[q];
    for (int t0 = wave * 64; t0 < total; t0 += kWaves * 64) {
        int t = t0 + lane, q = 0;
        if (t < total) {
            while (t >= counts[q]) t -= counts[q++];
            settle_entry<D, D>(reinterpret_cast<uint64_t *>(lds + S::LISTS)[q * S::LIST + t], h.of, h.proj, NB, 0, h.map);
        }
    }
}

template <int NE, int D, int NB>
int launch(const NormRows &norm, long T, const int8_t *w, float scale, const HashOut &h, float *v, bool split, hipStream_t st) {
    using S = NormHashShape<NE, D, NB>;
    const long blocks = (T + kRows - 1) / kRows, most = 256 * S::PER_CU;
    if (split)
        norm_hash_kernel<NE, D, NB, true><<<dim3((unsigned)(blocks * 3 * NE)), dim3(kWaves * 64), 0, st>>>(norm, T, w, scale, h, v);
    else
        norm_hash_kernel<NE, D, NB, false><<<dim3((unsigned)(blocks < most ? blocks : most)), dim3(kWaves * 64), 0, st>>>(norm, T, w, scale, h, v);
    return check_launch("LayerNorm, QKV projection and hash");
}

template <int NE>
int launch_width(const NormRows &norm, long T, const int8_t *w, float scale, const HashOut &h, int d, int nbits, float *v, bool split, hipStream_t st) {
    if (d == 32) return launch<NE, 32, 64>(norm, T, w, scale, h, v, split, st);
    return nbits == 64    ? launch<NE, 64, 64>(norm, T, w, scale, h, v, split, st)
           : nbits == 128 ? launch<NE, 64, 128>(norm, T, w, scale, h, v, split, st)
                          : launch<NE, 64, 256>(norm, T, w, scale, h, v, split, st);
}

}  // namespace

// A workgroup does 64 rows of everything one after the other, with one of it on a CU (two at E = 64 with heads of 32).  Separate launches
// spread a call finer: over columns of Wqkv and over bits of the hash.  Whole layers (linear attention, MLP of 4E; E = 256: 512), us with
// two launches and one:
//   E =  64         64 bits: 197 rows 22.7, 20.1; 16384 32.5, 29.1; 131072 94.3, 81.2 (heads of 64: 93.4, 89.2)
//                  256 bits: 197 rows 32.5, 31.6; 16384 48.3, 42.1; 20000 51.4, 51.3; 131072 132.8, 130.1
//   E = 128 .. 256, up to 256 workgroups, 64 bits: (128) 1576 rows 36.1, 35.0; 10400 45.4, 40.0; (256) 16384 74.2, 69.3
//                  128 bits: (128) 1576 rows 41.8, 42.2; 3152 43.5, 42.5; (192) 10400 65.1, 65.1; (256) 16384 86.5, 79.8
//                  256 bits: (128) 1576 rows 45.1, 48.3; 10400 56.4, 56.7; 13900 59.0, 57.1; (192) 10400 73.9, 76.8; 12000 80.5, 80.0;
//                            (256) 16384 102.4, 96.7
//   beyond, rounds of workgroups that take long lose more than the traffic saved (128, 20000 rows of 64 bits 58.1 with two launches) until
//   Q, K and V outgrow the cache behind L2: 64 bits (128) 95000 rows 156.6, 159.8; 100000 184.7, 182.7; 131072 229.2, 196.3.  Wider rows go
//   to linear_hash.hip there (192: 65536 rows 185.3, 179.0; 256: 100000 rows 419.7, 388.9), as do few of them that this does not take.
//
// Few rows: a workgroup for every 64 columns of Wqkv of 64 rows, all of which normalise the same rows and none of which does more than
// one chunk.  Up to one for every CU, and more where two share one (64 bits: E = 64, and 128 with heads of 32) or where the other ways are
// slow enough for a second or third round: the LDS is that of the walking kernels, so that with heads of 64 and 128 columns or more (82 KB
// and up) a CU has one at a time.  What takes the call otherwise (two or three launches, or one with all chunks), and this, us:
//   E =  64   64 bits: 197 rows 19.5, 18.1; 5600 25.7, 24.7; 10922 27.3, 26.4; 13000 27.7, 28.1.  256 bits: 197 rows 32.1, 29.6; 5440 36.9,
//            34.3; 8000 38.3, 40.1
//   E = 128   64 bits: 197 rows 30.5, 25.3; 2730 38.0, 32.3; 5600 39.1, 38.4; 6400 39.0, 40.1, heads of 32 37.0, 34.8.  128 bits: 5600 rows
//            44.4, 42.7; 8000 45.4, 49.9.  256 bits: 197 rows 39.5, 36.0; 3500 48.7, 45.4; 4096 47.1, 48.4
//   E = 192   64 bits: 197 rows 34.6, 31.8; 1792 41.4, 37.6; 1856 41.6, 43.3.  256 bits: 197 rows 43.5, 42.8; 1792 55.5, 49.7; 1856 55.0, 55.5
//   E = 256   64 bits: 49 rows 32.2, 28.9; 1344 43.3, 38.0; 1576 43.4 (linear_hash.hip), 45.5.  256 bits: 1344 rows 57.2, 50.5; 1700 57.9, 55.7
static bool by_chunks(long T, int E, int d, int nbits) {
    int most = 256;
    if (nbits == 64 && E == 64) most = 512;
    if (E == 128) most = nbits == 256 ? 336 : d == 32 ? 640 : 544;
    if (E == 256 && nbits == 256) most = 320;
    return (T + kRows - 1) / kRows * (3 * E / 64) <= most;
}

bool sa::norm_hash_one_launch(long T, int E, int H, int nbits) {
    const int d = E / H;
    if (!((d == 32 && nbits == 64) || (d == 64 && (nbits == 64 || nbits == 128 || nbits == 256)))) return false;
    if (E > 256 || E % 64 != 0 || T * H >= (1L << 31)) return false;
    if (by_chunks(T, E, d, nbits)) return true;
    if (!norm_linear_one_launch(T, E)) return false;
    if (E == 64) return true;
    if (T <= 256 * kRows) return nbits == 64 || T >= (nbits == 128 ? 3072 : 12288);
    return E == 128 && nbits == 64 && T * E >= 3L << 22;
}

int sa::launch_norm_hash(const NormRows &norm, int B, int N, int H, int E, const int8_t *wqkv_planes, float scale, const float *proj, int nbits,
                         float *q, float *k, uint64_t *q_codes, uint64_t *k_codes, float *v, hipStream_t st) {
    const HashOut h{proj, q, k, Tensors{q, k, q_codes, k_codes}, RowMap{FastDiv((uint32_t)H), FastDiv((uint32_t)N), N, H, nbits / 64}};
    const long T = (long)B * N;
    const bool split = by_chunks(T, E, E / H, nbits);
    switch (E) {
        case 64: return launch_width<1>(norm, T, wqkv_planes, scale, h, E / H, nbits, v, split, st);
        case 128: return launch_width<2>(norm, T, wqkv_planes, scale, h, E / H, nbits, v, split, st);
        case 192: return launch_width<3>(norm, T, wqkv_planes, scale, h, E / H, nbits, v, split, st);
        case 256: return launch_width<4>(norm, T, wqkv_planes, scale, h, E / H, nbits, v, split, st);
    }
    return fail(SA_ERR_UNSUPPORTED, "layer: width %d with the hash in the projection", E);
}
