// Both layers of a Shift MLP in one kernel, for widths whose output row a workgroup can hold (E = 64 .. 256):
//     y[row] = scale * W2 . lut[requant(W1 . x[row])]
// The hidden rows never leave the CU: 128 of their columns at a time are made from the rows of x (in registers), go through
// the table into LDS and are multiplied into the output, while the next 128 are made.  As two launches the MLP wrote and read
// them (134 MB for 131072 rows of 1024), and a tile of either spent as long on its way in and out as on its products (256 x 128
// of 1024 <- 256: 3.5 us of products in 10.4).  Both planes of both weights stream past, through a ring of three stages.
//
// Bound by how closely the two wavefronts of a SIMD pack products and the requantiser's vector operations (at E = 256 the matrix
// pipe is busy for half of a round); the weights, from the L2, are there in time.  Measured, two launches -> one:
//      25088 x  64, 512 hidden   20.0 -> 10.1 us     131072 x  64   49 -> 33
//      25088 x 192, 768 hidden   30 -> 24            131072 x 192  112 -> 93
//      16384 x 256, 1024 hidden  31 -> 26            131072 x 256  161 -> 145
// A layer's LayerNorm in front of it costs a workgroup its rows as fp32, asked for ahead of the first weights, and 4 MI of them per
// wavefront to normalise, and saves the launch that wrote the codes: layer of 32 x 784 tokens x 64 52.1 -> 47.1 us, of 1 x 16384
// x 256 122 -> 115.  With prepared weights the output projection in front of the LayerNorm is made here too, from all of Wo in
// LDS: at E = 64 it costs this launch 0.5 us and saves one of 5.7 (layer 47.1 -> 42.1 us), at E = 256 7.4 of 9.4 (121.9 -> 120.6).
// The loads of a stage go between the products that end the stage before: all of them ahead of those products, the wavefronts, which
// have just met, all waited for the memory pipe with the matrix cores idle (16384 x 256: 2.07 -> 1.77 us per 128 hidden columns of both
// layers, 4400 -> 3700 cycles of a CU whose matrix cores need 2048 for them; 131072 x 256, 1024 hidden 138.9 -> 128.1 us).  Of short hidden
// layers a workgroup of 128 rows takes tile after tile, the next one's weights and rows on their way while the outputs leave (launch_shift_mlp).
// The clock takes part of that back (2.14 -> 2.1 GHz: the card's power, not its issue slots, is what this kernel runs out of); layer of
// 16384 x 256 113.2 -> 111.1, of 32 x 784 x 64 39.8 -> 39.4.  Products of 32 x 32 x 32 needed a tenth fewer cycles and took the same time at
// 1.98 GHz, and the kernels around them longer (block of 8 x 16384 tokens 369 against 365).
// Layer 1 on four wavefronts and layer 2 on the other four (requantiser beside products without being interleaved): 226 us
// for the last one.
#include "common.h"
#include "gemm_common.h"
#include "gemm_mfma.h"
#include "gemm_stores.h"
#include "layernorm.h"

namespace {

using namespace sa;

typedef int v4i __attribute__((ext_vector_type(4)));

__device__ inline v4i mma16(const uint4 &a, const uint4 &b, v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, a), __builtin_bit_cast(v4i, b), c, 0, 0, 0);
}

constexpr int kMlpWaves = 8, kHidChunk = 128;

// NE: E / 64.  MI: 16-row tiles of a wavefront; the eight wavefronts stand 2 x 4 over rows x columns.  PROJECT: the rows are made here.
template <int NE, int MI, bool PROJECT, bool WALK, class Store>
struct MlpShape {
    static constexpr int E = 64 * NE, BM = 32 * MI;
    static constexpr int PS = NE <= 2 ? 2 : 1;               // planes of a stage
    static constexpr int SPG = 2 / PS;                       // stages of one layer of a chunk
    static constexpr int PLANE = kHidChunk * E;              // W1: 128 rows of E bytes; W2: E rows of 128 bytes
    static constexpr int STAGE = PS * PLANE, RING = 3, LOADS = PS * NE;
    static constexpr int PITCH = 64 * NE + 16;               // a staged output row of a wavefront's columns
    // (the table first: its offset is part of the instructions that read it)
    static constexpr int TABLE = 0, STAGES = 1024, H = STAGES + RING * STAGE, H_BYTES = BM * kHidChunk;
    static constexpr int WO_END = PROJECT ? STAGES + 2 * E * E : 0;      // Wo's planes, in the place of the stages and the hidden rows
    static constexpr int SIDE = H + 2 * H_BYTES > WO_END ? H + 2 * H_BYTES : WO_END;
    static constexpr int LDS_BYTES = SIDE + (WALK ? 2 : 1) * OutSide<Store, BM>::BYTES;
    static_assert(BM * E <= 2 * H_BYTES, "codes of normalised rows in the place of the hidden rows");
    static_assert(BM * E * 4 <= RING * STAGE + 2 * H_BYTES, "projected rows in the place of the ring and the hidden rows");
    static_assert(kMlpWaves * 16 * PITCH <= RING * STAGE, "output staging reuses the ring");
    static_assert(SIDE >= WO_END && LDS_BYTES <= 160 * 1024, "what the outputs read is fetched before Wo; LDS of a CU");
};

__device__ inline int swizzle_128(int r, int c) { return c ^ ((r >> 1) & 7); }

// What the rows are: codes; fp32 rows, which every wavefront normalises its share of; or fp32 rows that the kernel makes first, as
// x_res + Wo . codes.
enum MlpRows { kCodes, kNorm, kProject };

// A stage of weights: of which layer (0: none; 3: of the first, behind its last chunk the last of the second), which of its parts,
// and of which chunk.  Not live: nothing is loaded.
template <int LAYER, int SUB>
struct MlpStage {
    static constexpr int kLayer = LAYER, kSub = SUB;
    int chunk;
    bool live = true;
};

// WALK: a workgroup takes tile after tile (codes of 128 rows, more tiles than CUs).  A kernel of its own: what a workgroup keeps for the next
// tile costs one that has none (one tile a workgroup, prepared weights, one way out of this code and the other: 128 x 512, 16400
// rows 13.7 and 12.4 us, 128 x 768 17.9 and 15.9, 192 x 768 21.8 and 19.6, 256 x 1024, 32768 rows 35.5 and 33.2).
template <int NE, int MI, int ROWS, bool WALK, class Store>
__device__ __forceinline__ void shift_mlp_tiles(const int8_t *__restrict__ x, NormRows norm, RowSel sel, int hid,
                                                const int8_t *__restrict__ w1, const int8_t *__restrict__ w2,
                                                const int8_t *__restrict__ lut, float rq, Store store) {
    constexpr bool NORM = ROWS != kCodes, PROJECT = ROWS == kProject;
    using S = MlpShape<NE, MI, PROJECT, WALK, Store>;
    constexpr int E = S::E, PS = S::PS, SPG = S::SPG, LOADS = S::LOADS;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[S::LDS_BYTES];
    const int32_t *rows;
    long n_rows;
    resolve_rows(sel, rows, n_rows);
    long m0 = (long)blockIdx.x * S::BM;
    if (m0 >= n_rows) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 2, wc = wave & 3, fr = lane & 15, fg = lane >> 4;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    const int chunks = hid / kHidChunk;

    typedef OutSide<Store, S::BM> Side;
    Side side{store, rows, m0, n_rows, lds + S::SIDE};
    side.fetch_rows(wave, lane);
    if (wave == kMlpWaves - 1) direct_load_4(lut + lane * 4, lds_base + S::TABLE);

    v4i acc1[MI][2], acc2[MI][NE];
    auto clear = [&](v4i (&a)[MI][NE]) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int t = 0; t < NE; ++t) a[i][t] = v4i{0, 0, 0, 0};
    };
    // this wavefront's rows of x, as operands of the first layer (PROJECT: of the projection, until then)
    uint4 xf[MI][NE];
    constexpr int LPR = NE == 1 ? 16 : NE == 2 ? 32 : 64, GROUPS = 64 / LPR, STEPS = 4 * MI / GROUPS;      // NORM: lanes of a row
    const int l = lane % LPR, norm_row = wave * 4 * MI + lane / LPR;          // this lane's columns 4 l .. + 3 of rows norm_row + GROUPS i
    float4 xr[NORM ? STEPS : 1], gamma, beta;
    if constexpr (NORM) {
        const int col = min(4 * l, E - 4);                   // (lanes past the row: its end, not used; see row_or_zero)
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const long m = min(m0 + norm_row + GROUPS * i, n_rows - 1);
            xr[i] = *reinterpret_cast<const float4 *>((PROJECT ? norm.residual : norm.x) + (size_t)m * E + col);
        }
        gamma = *reinterpret_cast<const float4 *>(norm.gamma + col);
        beta = *reinterpret_cast<const float4 *>(norm.beta + col);
    }
    auto load_rows = [&](int of_lane, auto &&row_of) {       // row_of: which row of x is row ml of the tile
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int8_t *from = x + (size_t)row_of(wr * 16 * MI + 16 * i + (of_lane & 15)) * E + 16 * (of_lane >> 4);
#pragma unroll
            for (int k = 0; k < NE; ++k) xf[i][k] = *reinterpret_cast<const uint4 *>(from + 64 * k);
        }
    };
    if constexpr (ROWS != kNorm) {
        load_rows(lane, [&](int ml) { return rows ? (long)rows[side.row(ml)] : side.row(ml); });
    }

    if constexpr (PROJECT) {
        // Wo's planes in the place of all that comes later, the products as those of the second layer, through LDS to the
        // wavefronts that normalise the rows.
#pragma unroll
        for (int j = 0; j < NE * NE; ++j) {                  // 8 NE^2 KiB: the planes are one behind the other
            const int q = j * kMlpWaves + wave, c = q * 64 + lane, r = c / (4 * NE);
            direct_load_16(norm.wo, (uint32_t)(r * E + swizzle_row<NE>(r, c % (4 * NE)) * 16), lds_base + S::STAGES + q * 1024);
        }
        clear(acc2);
        wait_loads_in_flight<0>();
        __syncthreads();
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < NE; ++k)
#pragma unroll
                for (int t = 0; t < NE; ++t) {
                    const int r = p * E + wc * 16 * NE + 16 * t + fr;
                    const uint4 w = *reinterpret_cast<const uint4 *>(lds + S::STAGES + r * E + swizzle_row<NE>(r, 4 * k + fg) * 16);
#pragma unroll
                    for (int i = 0; i < MI; ++i) acc2[i][t] = mma16(w, xf[i][k], acc2[i][t]);
                }
        __syncthreads();                                     // Wo has been read
        auto staged = [&](int r, int c) { return reinterpret_cast<float4 *>(lds + S::STAGES + r * E * 4 + (c ^ (r & 15)) * 16); };
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int t = 0; t < NE; ++t)
                *staged(wr * 16 * MI + 16 * i + fr, wc * 4 * NE + 4 * t + fg) =
                    make_float4((float)acc2[i][t][0], (float)acc2[i][t][1], (float)acc2[i][t][2], (float)acc2[i][t][3]);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const int r = norm_row + GROUPS * i;
            if (4 * l < E) {
                const float4 a = *staged(r, l);
                xr[i] = make_float4(__builtin_fmaf(a.x, norm.scale, xr[i].x), __builtin_fmaf(a.y, norm.scale, xr[i].y),
                                    __builtin_fmaf(a.z, norm.scale, xr[i].z), __builtin_fmaf(a.w, norm.scale, xr[i].w));
                if (m0 + r < n_rows) *reinterpret_cast<float4 *>(norm.out + (size_t)(m0 + r) * E + 4 * l) = xr[i];
            }
        }
        __syncthreads();                                     // the ring's place is free
    }

    // Where this lane's 16 bytes of load i of a plane come from: a part that is the same in every lane (row0 rows) and one per
    // lane, whose chunk is flipped by `flip` bytes between the loads.
    const uint32_t lane2 = (uint32_t)(lane >> 3) * (uint32_t)hid + (uint32_t)((lane & 7) ^ (lane >> 4)) * 16;
    uint32_t lane1[NE == 3 ? 3 : 1];
    if constexpr (NE == 3) {
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int q = (wave * NE + i) * 64 + lane, r = q / (4 * NE);
            lane1[i] = (uint32_t)(r * E + swizzle_row<NE>(r, q % (4 * NE)) * 16);
        }
    } else {
        const int r = lane / (4 * NE);
        lane1[0] = (uint32_t)(r * E + swizzle_row<NE>(r, lane % (4 * NE)) * 16);
    }
    // The stages in the order they are multiplied: layer 1 of chunk 0, then layer 1 of chunk c + 1 before layer 2 of chunk c.  A
    // stage's loads go to the ring's place `to`, one at a time: back to back they would hold up the products.
    auto load_stage_of = [&](auto stage, int to, int j) {
        constexpr int LAYER = decltype(stage)::kLayer, SUB = decltype(stage)::kSub;
        const int p = j / NE, i = j % NE;
        uint32_t from = LAYER == 2 ? lane2 : lane1[NE == 3 ? i : 0];
        int w = wave;
        if constexpr (WALK && NE > 2) {                      // made here: no registers for every load's part of it (at E = 128 there are)
            asm volatile("" : "+v"(from), "+s"(w));
            w = __builtin_amdgcn_readfirstlane(w);
        }
        const int q = w * NE + i;
        const size_t plane = (size_t)(SUB * PS + p) * hid * E;
        const uint32_t at = lds_base + S::STAGES + to * S::STAGE + p * S::PLANE + q * 1024;
        if constexpr (LAYER == 2) {
            direct_load_16(w2 + plane + (size_t)stage.chunk * kHidChunk + (size_t)(q * 8) * hid, from ^ (q % 2 * 64), at);
        } else if constexpr (LAYER == 1) {
            const int8_t *base = w1 + plane + (size_t)stage.chunk * kHidChunk * E;
            if constexpr (NE == 3) direct_load_16(base, from, at);
            else direct_load_16(base + q * 1024, from ^ (NE == 4 ? i * 64 : NE == 2 ? q % 2 * 64 : 0), at);
        }
    };
    auto load_stage = [&](auto stage, int to, int j) {
        constexpr int LAYER = decltype(stage)::kLayer, SUB = decltype(stage)::kSub;
        if constexpr (LAYER == 3) {
            if (stage.chunk < chunks) load_stage_of(MlpStage<1, SUB>{stage.chunk}, to, j);
            else load_stage_of(MlpStage<2, SUB>{chunks - 1}, to, j);
        } else if (stage.live) {
            load_stage_of(stage, to, j);
        }
    };
    auto load_whole_stage = [&](auto stage, int to) {
#pragma unroll
        for (int j = 0; j < LOADS; ++j) load_stage(stage, to, j);
    };
    load_whole_stage(MlpStage<1, 0>{0}, 0);
    if constexpr (SPG == 2) {
        load_whole_stage(MlpStage<1, SPG - 1>{0}, 1);
        load_whole_stage(MlpStage<1, 0>{1}, 2);
    } else {
        load_whole_stage(MlpStage<1, 0>{1}, 1);
        load_whole_stage(MlpStage<2, 0>{0}, 2);
    }
    if constexpr (NORM) {                                    // the codes, by way of the hidden rows' place
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const float4 v[1] = {row_or_zero(xr[i], 4 * l < E)};
            float mean, rstd, y[4];
            row_stats<LPR, 1>(v, l, E, norm.eps, mean, rstd);
            normalise(v[0], mean, rstd, gamma, beta, y);
            const int r = norm_row + GROUPS * i;
            if (4 * l < E) *reinterpret_cast<uint32_t *>(lds + S::H + r * E + swizzle_row<NE>(r, l / 4) * 16 + l % 4 * 4) = codes_of(y, norm.inv_scale);
        }
    }
    wait_loads_in_flight<(S::RING - 1) * LOADS>();
    side.fetch_gates(wave, lane);
    __syncthreads();
    if constexpr (NORM) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int k = 0; k < NE; ++k) {
                const int r = wr * 16 * MI + 16 * i + fr;
                xf[i][k] = *reinterpret_cast<const uint4 *>(lds + S::H + r * E + swizzle_row<NE>(r, 4 * k + fg) * 16);
            }
        wait_lds_reads();                                    // hidden rows come here behind the first layer's barriers
    }
    int slot = 0;                                            // the place in the ring of the stage being multiplied

    // Operands are read one step ahead of their products.  A step is 64 k, in layer 1 of E = 128 and 256 two of them:
    // the products of one do not cover the latency of the LDS.  fb: weights, fa: hidden rows.
    constexpr int KS = NE % 2 == 0 ? 2 : 1;
    uint4 fb[2][4], fa[MI];
    // Addresses: the swizzles flip bits of a row's 16-byte chunks, and so does going along the contraction; tiles are whole rows apart.
    const uint32_t at1 = S::STAGES + (wc * 32 + fr) * E + swizzle_row<NE>(wc * 32 + fr, fg) * 16;
    const uint32_t at2 = S::STAGES + (wc * 16 * NE + fr) * kHidChunk + swizzle_128(wc * 16 * NE + fr, fg) * 16;
    const uint32_t at_h = S::H + (wr * 16 * MI + fr) * kHidChunk + swizzle_128(fr, fg) * 16;
    static_assert(S::STAGES % 256 == 0 && S::STAGE % 256 == 0 && S::H % 256 == 0, "the bits that are flipped are the rows' own");
    auto operand = [&](uint32_t at, uint32_t along, uint32_t tile) { return *reinterpret_cast<const uint4 *>(lds + ((at ^ along) + tile)); };
    auto read1 = [&](int par, int n) {                       // step n of a stage
        const uint32_t stage = at1 + slot * S::STAGE;
#pragma unroll
        for (int q = 0; q < KS; ++q)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int p = (n * KS + q) / NE, k = (n * KS + q) % NE;
                fb[par][2 * q + t] = NE == 3 ? operand(stage, 0, 64 * k + p * S::PLANE + 16 * t * E) : operand(stage, 64 * k, p * S::PLANE + 16 * t * E);
            }
    };
    auto read2 = [&](int par, int p, int k) {
        const uint32_t stage = at2 + slot * S::STAGE;
#pragma unroll
        for (int t = 0; t < NE; ++t) fb[par][t] = operand(stage, 64 * k, p * S::PLANE + 16 * t * kHidChunk);
    };
    auto hidden_at = [&](uint32_t at, int buf) {
        if constexpr (WALK && NE > 2) asm volatile("" : "+v"(at));     // made here: no registers from tile to tile for either buffer's
        return at + buf * S::H_BYTES;
    };
    auto read_hidden = [&](int i, int k, int buf) { fa[i] = operand(hidden_at(at_h, buf), 64 * k, 16 * i * kHidChunk); };
    // Before the last products of a stage, whose operands are in registers by then: the next stage is there (the one behind it need
    // not be), and the place of this one is free for the stage three ahead, whose loads go between those products.
    auto hand_over = [&](bool behind) {
        if (behind) wait_loads_in_flight<LOADS>();
        else wait_loads_in_flight<0>();
        __syncthreads();
        slot = slot == S::RING - 1 ? 0 : slot + 1;
    };
    auto left = [&]() { return slot == 0 ? S::RING - 1 : slot - 1; };
    enum { kNone, kLayer1, kLayer2 };
    // behind product u of N: its share of the stage's loads
    auto between = [&](auto u_c, auto n_c, auto stage) {
        constexpr int u = decltype(u_c)::value, N = decltype(n_c)::value;
        if constexpr (decltype(stage)::kLayer != 0) {
#pragma unroll
            for (int j = u * LOADS / N; j < (u + 1) * LOADS / N; ++j) {
                __builtin_amdgcn_sched_barrier(0);
                load_stage(stage, left(), j);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    auto first_of = [&](auto next_c) {              // the first operands of what comes next
        constexpr int next = decltype(next_c)::value;
        if constexpr (next == kLayer1) read1(0, 0);
        if constexpr (next == kLayer2) read2(0, 0, 0);
    };

    // Products are computed transposed (weights down, rows across): a lane holds four consecutive columns of row lane % 16.
    // buf: the hidden rows that a layer 2 behind this one reads; ahead0, ahead1: the stages to load as this layer's are done.
    auto layer1 = [&](auto next_c, int buf, auto ahead0, auto ahead1) {
        constexpr int STEPS = PS * NE / KS, ALL = SPG * STEPS;       // of a stage, of the layer
        static_for<ALL>([&](auto n_c) {
            constexpr int n = decltype(n_c)::value, m = n + 1;
            static_assert(ALL % 2 == 0, "what comes next starts with buffer 0");
            if constexpr (m % STEPS != 0) {
                read1(m & 1, m % STEPS);
            } else {
                hand_over(true);
                if constexpr (m < ALL) read1(m & 1, 0);
                else first_of(next_c);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (m == ALL && decltype(next_c)::value == kLayer2)
#pragma unroll
                for (int i = 0; i < MI; ++i) read_hidden(i, 0, buf);
            static_for<KS * MI * 2>([&](auto u_c) {
                constexpr int u = decltype(u_c)::value, i = u / (2 * KS), q = u / 2 % KS, t = u % 2;
                acc1[i][t] = mma16(fb[n & 1][2 * q + t], xf[i][(n * KS + q) % NE], n == 0 && q == 0 ? v4i{0, 0, 0, 0} : acc1[i][t]);
                if constexpr (m % STEPS == 0) {
                    if constexpr (m < ALL || SPG == 1) between(u_c, std::integral_constant<int, KS * MI * 2>{}, ahead0);
                    else between(u_c, std::integral_constant<int, KS * MI * 2>{}, ahead1);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // tile u % 2 of row tile u / 2 of the chunk's hidden columns: table entries, then a byte each into the hidden rows
    const uint32_t at_kept = S::H + (wr * 16 * MI + fr) * kHidChunk + swizzle_128(fr, wc * 2) * 16 + 4 * fg;
    auto lookup = [&](int u, uint32_t (&v)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = lds[S::TABLE + requant_index(acc1[u / 2][u % 2][r], rq)];
    };
    auto keep = [&](int u, const uint32_t (&v)[4], int buf) {
        *reinterpret_cast<uint32_t *>(lds + ((hidden_at(at_kept, buf) ^ (u % 2 * 16)) + 16 * (u / 2) * kHidChunk)) =
            (v[0] | (v[1] << 8)) | ((v[2] | (v[3] << 8)) << 16);
    };
    // Layer 2 of a chunk; between its products the next chunk's hidden columns go to the other buffer (requant), all of them
    // before the last step, whose barrier another layer 2 may read behind.
    // behind0, behind1: stages that may still be on their way when this layer's are done.
    auto layer2 = [&](int buf, auto requant_c, auto next_c, auto ahead0, auto ahead1, bool behind0, bool behind1) {
        constexpr bool REQUANT = decltype(requant_c)::value;
        constexpr int STEPS = PS * 2;
        uint32_t v[2][4];
        static_for<4>([&](auto n_c) {
            constexpr int n = decltype(n_c)::value, m = n + 1;
            if constexpr (m % STEPS != 0) {
                read2(m & 1, m % STEPS / 2, m % 2);
            } else {
                if constexpr (m < 4 || SPG == 1) hand_over(behind0);
                else hand_over(behind1);
                if constexpr (m < 4) read2(m & 1, 0, 0);
                else first_of(next_c);
            }
            __builtin_amdgcn_sched_barrier(0);
            static_for<MI * NE>([&](auto u_c) {
                constexpr int u = decltype(u_c)::value, i = u / NE, t = u % NE;
                acc2[i][t] = mma16(fb[n & 1][t], fa[i], acc2[i][t]);
                if constexpr (m % STEPS == 0) {
                    if constexpr (m < 4 || SPG == 1) between(u_c, std::integral_constant<int, MI * NE>{}, ahead0);
                    else between(u_c, std::integral_constant<int, MI * NE>{}, ahead1);
                }
                if constexpr (t == NE - 1) {
                    if constexpr (m < 4) read_hidden(i, m % 2, buf);
                    else if constexpr (decltype(next_c)::value == kLayer2) read_hidden(i, 0, buf ^ 1);
                    if constexpr (REQUANT) {
                        constexpr int at = n * MI + i;       // the table's answers are used two places after they are asked for
                        if constexpr (at >= 2 && at - 2 < 2 * MI) keep(at - 2, v[at & 1], buf ^ 1);
                        if constexpr (at < 2 * MI) lookup(at, v[at & 1]);
                    }
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using Layer1 = std::integral_constant<int, kLayer1>;
    using Layer2 = std::integral_constant<int, kLayer2>;
    using None = std::integral_constant<int, kNone>;

    using NoStage = MlpStage<0, 0>;

    // The stages ahead are three further on: of two parts of a layer, or one.
    for (;;) {
    const long next_m0 = m0 + (long)gridDim.x * S::BM;
    const bool more = WALK && next_m0 < n_rows;
    const Side next_side{store, rows, next_m0, n_rows, lds + 2 * S::SIDE + Side::BYTES - (side.lds - lds)};      // the two take turns
    clear(acc2);
    read1(0, 0);
    if constexpr (SPG == 2) layer1(Layer1{}, 0, MlpStage<1, 1>{1}, MlpStage<2, 0>{0});
    else layer1(Layer1{}, 0, MlpStage<3, 0>{2}, NoStage{});
    if (more) {                                              // behind a barrier that the outputs of the tile before are before
        int of_lane = lane;
        asm volatile("" : "+v"(of_lane));
        next_side.fetch_rows(wave, of_lane);
    }
    {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 2 * MI; ++u) {
            lookup(u, v);
            keep(u, v, 0);
        }
    }
    for (int c = 0; c + 2 < chunks; ++c) {
        if constexpr (SPG == 2) {
            layer1(Layer2{}, c & 1, MlpStage<2, 1>{c}, MlpStage<1, 0>{c + 2});
            layer2(c & 1, std::true_type{}, Layer1{}, MlpStage<1, 1>{c + 2}, MlpStage<2, 0>{c + 1}, true, true);
        } else {
            layer1(Layer2{}, c & 1, MlpStage<2, 0>{c + 1}, NoStage{});
            layer2(c & 1, std::true_type{}, Layer1{}, MlpStage<3, 0>{c + 3}, NoStage{}, true, true);
        }
    }
    if constexpr (SPG == 2) {
        layer1(Layer2{}, chunks & 1, MlpStage<2, 1>{chunks - 2}, MlpStage<2, 0>{chunks - 1});
        layer2(chunks & 1, std::true_type{}, Layer2{}, MlpStage<2, 1>{chunks - 1}, MlpStage<1, 0>{0, more}, true, true);
        layer2((chunks & 1) ^ 1, std::false_type{}, None{}, MlpStage<1, 1>{0, more}, MlpStage<1, 0>{1, more}, more, more);
    } else {
        layer1(Layer2{}, chunks & 1, MlpStage<1, 0>{0, more}, NoStage{});
        layer2(chunks & 1, std::true_type{}, Layer2{}, MlpStage<1, 0>{1, more}, NoStage{}, more, more);
        layer2((chunks & 1) ^ 1, std::false_type{}, None{}, MlpStage<2, 0>{0, more}, NoStage{}, more, more);
    }
    int out_lane = lane;
    asm volatile("" : "+v"(out_lane));                       // addresses of the outputs are made here, not kept from tile to tile
    if (more) {                                              // (in time behind the outputs)
        next_side.fetch_gates(wave, out_lane);
        load_rows(out_lane, [&](int ml) { return next_side.dest(ml); });
    }

    // ---- rows out, 16 of the wavefront's columns at a time, through LDS of its own: in the place of the hidden rows where the ring
    //      already has the next tile's weights
    if constexpr (!WALK) __syncthreads();                    // the ring has been read (the last stage's hand-over says so of the hidden rows)
    constexpr int OUT_COLS = WALK && NE % 2 == 0 ? 32 : 16 * NE, PARTS = 16 * NE / OUT_COLS, OUT_CHUNKS = OUT_COLS / 4;
    constexpr bool SWIZZLE = OUT_CHUNKS == 8;                // whole lines of the LDS: no room for a pitch
    constexpr int OUT_PITCH = SWIZZLE ? OUT_COLS * 4 : S::PITCH;
    static_assert(kMlpWaves * 16 * OUT_PITCH <= (WALK ? 2 * S::H_BYTES : S::RING * S::STAGE), "room for the outputs");
    uint8_t *slab = lds + (WALK ? S::H : S::STAGES) + wave * 16 * OUT_PITCH;
    auto staged_out = [&](int row, int c) { return reinterpret_cast<uint4 *>(slab + row * OUT_PITCH + (SWIZZLE ? c ^ (row & 7) : c) * 16); };
    constexpr int NC = OUT_CHUNKS / 4;                       // 16-byte chunks of a lane per part of 16 rows
    const int out_fr = out_lane & 15, out_fg = out_lane >> 4;
    auto place = [&](int j, int &row, int &c) {              // chunk j of this lane
        const int q = j * 64 + out_lane;
        row = q / OUT_CHUNKS;
        c = q % OUT_CHUNKS;
    };
    auto out_col = [&](int part, int c) { return wc * 16 * NE + part * OUT_COLS + 4 * c; };
    auto emit = [&](auto reads_c) {
        constexpr bool READS = decltype(reads_c)::value;
        float4 ext[READS ? 2 : 1][NC];
        auto fetch = [&](int n) {
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                int row, c;
                place(j, row, c);
                ext[READS ? n & 1 : 0][j] = READS ? ChunkOut<Store>(store, out_col(n % PARTS, c), E).fetch(side.dest(wr * 16 * MI + 16 * (n / PARTS) + row))
                                                  : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        };
        fetch(0);
#pragma unroll
        for (int n = 0; n < MI * PARTS; ++n) {
            const int i = n / PARTS, part = n % PARTS;
            if (n + 1 < MI * PARTS) fetch(n + 1);
#pragma unroll
            for (int t = 0; t < NE / PARTS; ++t) {
                const v4i &a = acc2[i][part * (NE / PARTS) + t];
                uint32_t w[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) w[r] = store.convert(a[r], 0, nullptr);
                *staged_out(out_fr, 4 * t + out_fg) = make_uint4(w[0], w[1], w[2], w[3]);
            }
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                int row, c;
                place(j, row, c);
                const uint4 v = *staged_out(row, c);
                const int ml = wr * 16 * MI + 16 * i + row;
                if (m0 + ml < n_rows) ChunkOut<Store>(store, out_col(part, c), E).put(v, ext[READS ? n & 1 : 0][j], side.gate(ml), side.dest(ml));
            }
        }
    };
    if (store.accumulate) emit(std::true_type{});
    else emit(std::false_type{});
    if (!more) return;
    m0 = side.m0 = next_m0;
    side.lds = next_side.lds;
    }
}

template <int NE, int MI, int ROWS, class Store>
__global__ __launch_bounds__(kMlpWaves * 64) void shift_mlp_kernel(const int8_t *__restrict__ x, NormRows norm, RowSel sel, int hid,
                                                                   const int8_t *__restrict__ w1, const int8_t *__restrict__ w2,
                                                                   const int8_t *__restrict__ lut, float rq, Store store) {
    shift_mlp_tiles<NE, MI, ROWS, false>(x, norm, sel, hid, w1, w2, lut, rq, store);
}

template <int NE, class Store>
__global__ __launch_bounds__(kMlpWaves * 64) void shift_mlp_walk_kernel(const int8_t *__restrict__ x, RowSel sel, int hid,
                                                                        const int8_t *__restrict__ w1, const int8_t *__restrict__ w2,
                                                                        const int8_t *__restrict__ lut, float rq, Store store) {
    shift_mlp_tiles<NE, 4, kCodes, true>(x, NormRows{}, sel, hid, w1, w2, lut, rq, store);
}

struct MlpArgs {
    const int8_t *x;
    const NormRows *norm;                                    // or null
    RowSel sel;
    int hid;
    const int8_t *w1, *w2, *lut;
    float rq;
    ShiftStore<kEpiScatterI32> store;
};

// walk: 256 workgroups take the tiles one after the other
template <int NE, int MI>
int launch(const MlpArgs &a, bool walk, hipStream_t st) {
    typedef ShiftStore<kEpiScatterI32> Store;
    const long blocks = (a.sel.max_rows + 32 * MI - 1) / (32 * MI);
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_shift_mlp: too many rows for one launch");
    const dim3 grid((unsigned)blocks), block(kMlpWaves * 64);
    if (a.norm && a.norm->wo)
        shift_mlp_kernel<NE, MI, kProject, Store><<<grid, block, 0, st>>>(a.x, *a.norm, a.sel, a.hid, a.w1, a.w2, a.lut, a.rq, a.store);
    else if (a.norm)
        shift_mlp_kernel<NE, MI, kNorm, Store><<<grid, block, 0, st>>>(nullptr, *a.norm, a.sel, a.hid, a.w1, a.w2, a.lut, a.rq, a.store);
    else if (!walk)
        shift_mlp_kernel<NE, MI, kCodes, Store><<<grid, block, 0, st>>>(a.x, NormRows{}, a.sel, a.hid, a.w1, a.w2, a.lut, a.rq, a.store);
    else if constexpr (MI == 4)
        shift_mlp_walk_kernel<NE, Store><<<dim3(256), block, 0, st>>>(a.x, a.sel, a.hid, a.w1, a.w2, a.lut, a.rq, a.store);
    return check_launch("sa_shift_mlp (both layers)");
}

}  // namespace

// Whether one launch is the faster way, from sweeps over 197 .. 131072 rows, 256 .. 1536 hidden columns (two launches, one; us).
//  * Few rows: a workgroup passes all weights through its CU, about 1 us per 128 hidden columns and 64 of E / 2, whatever its rows.
//    So for E = 64 and 128 with small products always (E * hid up to 96 Ki: 64 x 512, 1568 rows 11.8 and 9.1; layer of 33 x 128, 768
//    hidden 33.8 and 30.6), with wider rows from where a good part of the chip has some (layer of 192, 512 hidden: 2400 rows 46.5
//    and 48.2, 3152 rows 51.4 and 50.1; 256, 384 hidden: 1000 rows 42.1 and 46.2, 3152 rows 54.4 and 53.5), for larger products
//    once their rows fill half of it (192 x 768: 6304 rows 16.4 and 15.6, layer 60.4 and 57.2, on packed weights 61.5 and 61.4;
//    192 x 1024 layer 6304 rows 66.1 and 66.6), beyond 1024 hidden columns a little more (128 x 1536: 7168 rows 0.985, 9216 rows
//    1.39 times as fast in one), as for 256 columns (256 x 1024: 10500 rows 21.6 and 22.4, 11200 rows 22.4 and 22.6, 12000 rows 23.2
//    and 22.6, packed 24.1 and 26.0, 15000 rows 27.1 and 26.4), and beyond 1536 not before the chip is full of them (256 x 2048: 12000
//    rows 35.3 and 39.2, 15000 rows 39.6 both, 16384 rows 41.6 and 40.1; 192 x 2048: 10500 rows 29.6 and 32.6, 11200 rows 35.8 and 32.6).
//  * On packed weights one launch needs another that decodes them, where two layers decode for themselves: only with enough hidden
//    columns (12608 rows of 256: 384 hidden 0.93 times, 512 0.94, 640 0.98, 768 0.96, of 16384 1.00; of 128: 256 0.98, 512 1.10).
//  * Beyond 16384 rows a workgroup has 128 and a CU one workgroup, so the launch takes whole rounds of 32768 rows, and what the last
//    round lacks costs as much as what it has: 256 x 1024, 32768 rows 1.26 times as fast in one, 33000 rows (two rounds) 50.1 and
//    71.1, 40000 57.6 and 69.3, 53000 67.5 and 70.0, 57000 the same, 65536 1.10, 82000 (three) 98.6 and 100, 90000 1.06.  Narrower
//    rows stand more of it, as two launches take longer with them, and more rounds (192 x 768: 40000 rows 42.4 and 43.7, 48000 1.03,
//    76000 1.05; 128 x 512: 40000 22.9 and 25.3, 48000 1.01, 76000 1.13), and hidden columns that are no power of two, whose tiles
//    the two launches fill less well (128 x 768: 40000 rows 37.1 and 33.4; 256 x 768: 20000 rows 31.5 and 28.3, 256 x 1024 33.0 and
//    34.3).  On packed weights a little less.
//  * In a layer the LayerNorm's launch is saved as well: only a second round that is nearly empty costs more than that (33000 x 256,
//    1024 hidden 169.5 and 186.6, 40000 187.7 and 199.2 on packed weights, 44000 1.03; 40000 x 256, 1536 hidden 235 and 217; 33000 x
//    192, 768 hidden 145.9 and 156, 44000 1.01; 33000 x 128, 512 hidden 1.02; 70000 x 256, three rounds, 1.06).
//  * Of a row count that only the device knows any share of the bound may come, in one launch's rounds as in two launches: one only
//    where it is not the slower way for 30, 50, 70 and all of them (two launches / one, prepared weights).  128 x 512: 33000 rows
//    1.11, 1.54, 1.69, 1.21, 2000 rows 1.31 .. 1.25; 128 x 1536: 12608 rows 0.94, 1.08, 1.37, 1.57, 8000 rows 0.68 .. 1.26; on packed
//    weights 128 x 768: 17000 rows 1.00, 1.19, 1.42, 1.04, 8000 rows 0.91 .. 1.12.  Beyond 128 columns only small products up to one
//    round of 64 rows (192 x 384: 12608 rows 1.15, 1.25, 1.35, 1.77; 256 x 384 0.96, 1.10, 1.40, 1.66): 192 x 768, 12608 rows 0.84 ..
//    1.59, 33000 rows 0.85, 1.15, 1.52, 0.90; 256 x 1024, 17000 rows 0.55 .. 1.18; and on packed weights not at all (256 x 2048, 30 % of
//    26415 rows 65.2 us in one launch, 39.5 in two).
static bool counted_one_launch(long rows, int E, int hid, bool packed) {
    if (E <= 128) return (E == 64 || !packed || hid >= 384) && (hid <= (E == 64 ? 1536 : packed ? 512 : 768) || rows >= 96L * E);
    return !packed && (long)E * hid <= 98304 && rows >= 16L * E && rows <= 16384;
}

bool sa::shift_mlp_one_launch(const RowSel &sel, int E, int hid, MlpCall call) {
    if (E > 256 || E % 64 != 0 || hid % kHidChunk != 0 || hid < 2 * kHidChunk) return false;
    const long rows = sel.max_rows;
    if (sel.counts) return counted_one_launch(rows, E, hid, call == kMlpPacked);
    if ((long)E * hid > 98304 ? rows < 40L * E : E > 128 && rows < 16L * E) return false;
    if (E == 64) return true;
    if (call == kMlpPacked && hid < (E == 256 ? 640 : 384)) return false;
    if (call != kMlpInLayer) {
        if (hid >= 1024 && E == 256 && rows < (call == kMlpPacked ? 14000 : 11000)) return false;
        if (hid > 1536 && E > 128 && rows < (E == 256 ? 15000 : 11000)) return false;
        if (hid > 1024 && rows < 9000) return false;
    }
    if (rows <= 16384) return true;
    const long round = 32768, rounds = (rows + round - 1) / round, idle = 100 * (rounds * round - rows) / round;      // in % of a round
    const bool packed = call == kMlpPacked, power = (hid & (hid - 1)) == 0;
    if (call == kMlpInLayer) return E == 128 || rounds != 2 || idle <= (power ? 70 : 80);
    if (E == 128) return idle <= (power ? 35 : 50) + 15 * rounds;
    if (E == 256) return idle <= (packed ? 25 : rounds == 1 && !power ? 46 : 35);
    if (rounds == 1) return idle <= (packed ? 35 : 50);
    return idle <= (!packed ? 35 + 12 * rounds : hid < 768 ? 20 + 15 * rounds : 35 + 16 * rounds);
}

// Rows of a workgroup: 64, or 128 where that takes fewer rounds of the chip by more than the 1.45 times that a round of the
// larger ones takes (256 x 1024: 16384 rows 26 against 36 us, 25088 rows 47 against 37, 131072 rows 181 against 145).  At
// E = 64 two of the smaller share a CU (131072 rows 33 against 34 us).  Of rows that only the device counts half are expected.
// More of the larger ones than CUs: one after the other on 256 workgroups where the hidden layer is short.  What a tile saves is its start
// and its outputs' wait, and from 192 columns on every chunk pays for it with addresses made anew (a workgroup a tile / walking, us: 128 x
// 512, 131072 rows 48.3, 45.4; 128 x 1024 77.9, 75.2; 128 x 2048 131.8, 133.3; 192 x 256 44.9, 42.4; 192 x 384 54.6, 53.7; 192 x 768 82.5, 86.5;
// 256 x 512 82.3, 81.2; 256 x 768, 65536 rows 53.6, 55.2; 256 x 1024 65.1, 67.8, 131072 rows 127.8, 131.7).  By the bound of rows that only the
// device counts: with fewer after all walking costs 0.1 us (128 x 256, 30 % of 66000 rows 9.85, 10.0), with more it saves (all of 40000
// rows of 128 x 256 18.3, 16.0).
int sa::launch_shift_mlp(const int8_t *x, const NormRows *norm, const RowSel &sel, int E, int hid, const int8_t *w1_planes,
                         const int8_t *w2_planes, const int8_t *lut, float requant_scale, const Epilogue &out, hipStream_t st) {
    SA_REQUIRE(!norm || (!sel.rows && !out.gate), SA_ERR_INVALID, "sa_shift_mlp: rows to normalise are all rows, ungated");
    const MlpArgs a{x, norm, sel, hid, w1_planes, w2_planes, lut, requant_scale_finite(requant_scale), ShiftStore<kEpiScatterI32>(out)};
    const long m_est = sel.counts ? (sel.max_rows + 1) / 2 : sel.max_rows;
    auto rounds = [&](long rows) { return ((m_est + rows - 1) / rows + 255) / 256; };
    const bool tall = 29 * rounds(128) < 20 * rounds(64), walk = sel.max_rows > 256 * 128 && hid <= (E == 128 ? 1024 : E == 192 ? 384 : 512);
    switch (E) {
        case 64: return launch<1, 2>(a, false, st);
        case 128: return tall ? launch<2, 4>(a, walk, st) : launch<2, 2>(a, false, st);
        case 192: return tall ? launch<3, 4>(a, walk, st) : launch<3, 2>(a, false, st);
        case 256: return tall ? launch<4, 4>(a, walk, st) : launch<4, 2>(a, false, st);
    }
    return fail(SA_ERR_UNSUPPORTED, "sa_shift_mlp: width %d in one launch", E);
}
