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
template <int NE, int MI, bool PROJECT, class Store>
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
    static constexpr int LDS_BYTES = SIDE + OutSide<Store, BM>::BYTES;
    static_assert(BM * E <= 2 * H_BYTES, "codes of normalised rows in the place of the hidden rows");
    static_assert(BM * E * 4 <= RING * STAGE + 2 * H_BYTES, "projected rows in the place of the ring and the hidden rows");
    static_assert(kMlpWaves * 16 * PITCH <= RING * STAGE, "output staging reuses the ring");
    static_assert(SIDE >= WO_END && LDS_BYTES <= 160 * 1024, "what the outputs read is fetched before Wo; LDS of a CU");
};

__device__ inline int swizzle_128(int r, int c) { return c ^ ((r >> 1) & 7); }

// What the rows are: codes; fp32 rows, which every wavefront normalises its share of; or fp32 rows that the kernel makes first, as
// x_res + Wo . codes.
enum MlpRows { kCodes, kNorm, kProject };

template <int NE, int MI, int ROWS, class Store>
__global__ __launch_bounds__(kMlpWaves * 64) void shift_mlp_kernel(const int8_t *__restrict__ x, NormRows norm, RowSel sel, int hid,
                                                                   const int8_t *__restrict__ w1, const int8_t *__restrict__ w2,
                                                                   const int8_t *__restrict__ lut, float rq, Store store) {
    constexpr bool NORM = ROWS != kCodes, PROJECT = ROWS == kProject;
    using S = MlpShape<NE, MI, PROJECT, Store>;
    constexpr int E = S::E, PS = S::PS, SPG = S::SPG, LOADS = S::LOADS;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[S::LDS_BYTES];
    const int32_t *rows;
    long n_rows;
    resolve_rows(sel, rows, n_rows);
    const long m0 = (long)blockIdx.x * S::BM;
    if (m0 >= n_rows) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 2, wc = wave & 3, fr = lane & 15, fg = lane >> 4;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    const int chunks = hid / kHidChunk;

    const OutSide<Store, S::BM> side{store, rows, m0, n_rows, lds + S::SIDE};
    side.fetch_rows(wave, lane);
    if (wave == kMlpWaves - 1) direct_load_4(lut + lane * 4, lds_base + S::TABLE);

    v4i acc1[MI][2], acc2[MI][NE];
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
#pragma unroll
    for (int i = 0; i < (ROWS == kNorm ? 0 : MI); ++i) {
        const long m = min(m0 + wr * 16 * MI + 16 * i + fr, n_rows - 1);
        const int8_t *xr = x + (size_t)(rows ? (long)rows[m] : m) * E + 16 * fg;
#pragma unroll
        for (int k = 0; k < NE; ++k) xf[i][k] = *reinterpret_cast<const uint4 *>(xr + 64 * k);
    }

    if constexpr (PROJECT) {
        // Wo's planes in the place of all that comes later, the products as those of the second layer, through LDS to the
        // wavefronts that normalise the rows.
#pragma unroll
        for (int j = 0; j < NE * NE; ++j) {                  // 8 NE^2 KiB: the planes are one behind the other
            const int q = j * kMlpWaves + wave, c = q * 64 + lane, r = c / (4 * NE);
            direct_load_16(norm.wo, (uint32_t)(r * E + swizzle_row<NE>(r, c % (4 * NE)) * 16), lds_base + S::STAGES + q * 1024);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int t = 0; t < NE; ++t) acc2[i][t] = v4i{0, 0, 0, 0};
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
    // The stages in the order they are multiplied: layer 1 of chunk 0, then layer 1 of chunk c + 1 before layer 2 of chunk c.
    const int n_stages = 2 * chunks * SPG;
    auto issue = [&](int s, int slot) {
        const int u = s / SPG, sub = s % SPG;
        const bool second = u == 2 * chunks - 1 || (u > 0 && u % 2 == 0);
        const int c = u == 2 * chunks - 1 ? chunks - 1 : second ? u / 2 - 1 : (u + 1) / 2;
#pragma unroll
        for (int p = 0; p < PS; ++p) {
            const size_t plane = (size_t)(sub * PS + p) * hid * E;
            const uint32_t at = lds_base + S::STAGES + slot * S::STAGE + p * S::PLANE + wave * NE * 1024;
            if (second) {
                const int8_t *base = w2 + plane + (size_t)c * kHidChunk + (size_t)(wave * NE * 8) * hid;
#pragma unroll
                for (int i = 0; i < NE; ++i) direct_load_16(base + (size_t)i * 8 * hid, lane2 ^ ((wave * NE + i) % 2 * 64), at + i * 1024);
            } else {
                const int8_t *base = w1 + plane + (size_t)c * kHidChunk * E;
#pragma unroll
                for (int i = 0; i < NE; ++i) {
                    if constexpr (NE == 3) direct_load_16(base, lane1[NE == 3 ? i : 0], at + i * 1024);
                    else direct_load_16(base + (wave * NE + i) * 1024, lane1[0] ^ (NE == 4 ? i * 64 : NE == 2 ? (wave * NE + i) % 2 * 64 : 0), at + i * 1024);
                }
            }
        }
    };
#pragma unroll
    for (int q = 0; q < S::RING; ++q) issue(q, q);           // (there are at least four stages)
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
    int s = 0, slot = 0;                                     // the stage being multiplied, its place in the ring

#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int t = 0; t < NE; ++t) acc2[i][t] = v4i{0, 0, 0, 0};

    // Operands are read one step ahead of their products.  A step is 64 k, in layer 1 of E = 128 and 256 two of them:
    // the products of one do not cover the latency of the LDS.  fb: weights, fa: hidden rows.
    constexpr int KS = NE % 2 == 0 ? 2 : 1;
    uint4 fb[2][4], fa[MI];
    auto read1 = [&](int par, int n) {                       // step n of a stage
#pragma unroll
        for (int q = 0; q < KS; ++q)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int p = (n * KS + q) / NE, k = (n * KS + q) % NE, r = wc * 32 + 16 * t + fr;
                fb[par][2 * q + t] = *reinterpret_cast<const uint4 *>(lds + S::STAGES + slot * S::STAGE + p * S::PLANE + r * E + swizzle_row<NE>(r, 4 * k + fg) * 16);
            }
    };
    auto read2 = [&](int par, int p, int k) {
#pragma unroll
        for (int t = 0; t < NE; ++t) {
            const int r = wc * 16 * NE + 16 * t + fr;
            fb[par][t] = *reinterpret_cast<const uint4 *>(lds + S::STAGES + slot * S::STAGE + p * S::PLANE + r * kHidChunk + swizzle_128(r, 4 * k + fg) * 16);
        }
    };
    auto read_hidden = [&](int i, int k, int buf) {
        const int r = wr * 16 * MI + 16 * i + fr;
        fa[i] = *reinterpret_cast<const uint4 *>(lds + S::H + buf * S::H_BYTES + r * kHidChunk + swizzle_128(r, 4 * k + fg) * 16);
    };
    // Before the last products of a stage, whose operands are in registers by then: the next stage is there, and the place of
    // this one is free for the stage three ahead.
    auto hand_over = [&]() {
        if (s + 2 < n_stages) wait_loads_in_flight<LOADS>();
        else wait_loads_in_flight<0>();
        __syncthreads();
        if (s + S::RING < n_stages) issue(s + S::RING, slot);
        ++s;
        slot = slot == S::RING - 1 ? 0 : slot + 1;
    };
    enum { kNone, kLayer1, kLayer2 };
    auto first_of = [&](auto next_c) {              // the first operands of what comes next
        constexpr int next = decltype(next_c)::value;
        if constexpr (next == kLayer1) read1(0, 0);
        if constexpr (next == kLayer2) read2(0, 0, 0);
    };

    // Products are computed transposed (weights down, rows across): a lane holds four consecutive columns of row lane % 16.
    // buf: the hidden rows that a layer 2 behind this one reads.
    auto layer1 = [&](auto next_c, int buf) {
        constexpr int STEPS = PS * NE / KS, ALL = SPG * STEPS;        // of a stage, of the layer
        static_for<ALL>([&](auto n_c) {
            constexpr int n = decltype(n_c)::value, m = n + 1;
            static_assert(ALL % 2 == 0, "what comes next starts with buffer 0");
            if constexpr (m % STEPS != 0) {
                read1(m & 1, m % STEPS);
            } else {
                hand_over();
                if constexpr (m < ALL) read1(m & 1, 0);
                else first_of(next_c);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                if (m == ALL && decltype(next_c)::value == kLayer2) read_hidden(i, 0, buf);
#pragma unroll
                for (int q = 0; q < KS; ++q)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc1[i][t] = mma16(fb[n & 1][2 * q + t], xf[i][(n * KS + q) % NE], n == 0 && q == 0 ? v4i{0, 0, 0, 0} : acc1[i][t]);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // tile (i, t) of the chunk's hidden columns: table entries, then a byte each into the hidden rows
    auto lookup = [&](int i, int t, uint32_t (&v)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = lds[S::TABLE + requant_index(acc1[i][t][r], rq)];
    };
    auto keep = [&](int i, int t, const uint32_t (&v)[4], int buf) {
        const int r = wr * 16 * MI + 16 * i + fr, c = wc * 2 + t;
        *reinterpret_cast<uint32_t *>(lds + S::H + buf * S::H_BYTES + r * kHidChunk + swizzle_128(r, c) * 16 + 4 * fg) =
            (v[0] | (v[1] << 8)) | ((v[2] | (v[3] << 8)) << 16);
    };
    // Layer 2 of a chunk; between its products the next chunk's hidden columns go to the other buffer (requant), all of them
    // before the last step, whose barrier another layer 2 may read behind.
    auto layer2 = [&](int buf, auto requant_c, auto next_c) {
        constexpr bool REQUANT = decltype(requant_c)::value;
        constexpr int STEPS = PS * 2;
        uint32_t v[2][4];
        static_for<4>([&](auto n_c) {
            constexpr int n = decltype(n_c)::value, m = n + 1;
            if constexpr (m % STEPS != 0) {
                read2(m & 1, m % STEPS / 2, m % 2);
            } else {
                hand_over();
                if constexpr (m < 4) read2(m & 1, 0, 0);
                else first_of(next_c);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < MI; ++i) {
#pragma unroll
                for (int t = 0; t < NE; ++t) acc2[i][t] = mma16(fb[n & 1][t], fa[i], acc2[i][t]);
                if constexpr (m < 4) read_hidden(i, m % 2, buf);
                else if constexpr (decltype(next_c)::value == kLayer2) read_hidden(i, 0, buf ^ 1);
                if constexpr (REQUANT) {
                    const int at = n * MI + i;               // the table's answers are used two places after they are asked for
                    if (at >= 2 && at - 2 < 2 * MI) keep((at - 2) / 2, at % 2, v[at & 1], buf ^ 1);
                    if (at < 2 * MI) lookup(at / 2, at % 2, v[at & 1]);
                }
            }
            if constexpr (REQUANT && n < 3) {                // what a product's shadow holds behind each
#pragma unroll
                for (int q = 0; q < MI * NE; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 16 / NE, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using Layer1 = std::integral_constant<int, kLayer1>;
    using Layer2 = std::integral_constant<int, kLayer2>;
    using None = std::integral_constant<int, kNone>;

    read1(0, 0);
    layer1(Layer1{}, 0);
    {
        uint32_t v[4];
#pragma unroll
        for (int n = 0; n < 2 * MI; ++n) {
            lookup(n / 2, n % 2, v);
            keep(n / 2, n % 2, v, 0);
        }
    }
    for (int c = 0; c + 2 < chunks; ++c) {
        layer1(Layer2{}, c & 1);
        layer2(c & 1, std::true_type{}, Layer1{});
    }
    layer1(Layer2{}, chunks & 1);
    layer2(chunks & 1, std::true_type{}, Layer2{});
    layer2((chunks & 1) ^ 1, std::false_type{}, None{});

    // ---- rows out, 16 of the wavefront's columns at a time, through LDS of its own
    __syncthreads();                                         // the ring has been read
    uint8_t *slab = lds + S::STAGES + wave * 16 * S::PITCH;
    auto place = [&](int j, int &row, int &col) {            // chunk j of this lane: row of 16, first column
        const int q = j * 64 + lane;
        row = q / (4 * NE);
        col = wc * 16 * NE + q % (4 * NE) * 4;
    };
    auto emit = [&](auto reads_c) {
        constexpr bool READS = decltype(reads_c)::value;
        float4 ext[READS ? 2 : 1][NE];
        auto fetch = [&](int i) {
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                int row, col;
                place(j, row, col);
                ext[READS ? i & 1 : 0][j] =
                    READS ? ChunkOut<Store>(store, col, E).fetch(side.dest(wr * 16 * MI + 16 * i + row)) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        };
        fetch(0);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (i + 1 < MI) fetch(i + 1);
#pragma unroll
            for (int t = 0; t < NE; ++t) {
                uint32_t w[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) w[r] = store.convert(acc2[i][t][r], 0, nullptr);
                *reinterpret_cast<uint4 *>(slab + fr * S::PITCH + (16 * t + 4 * fg) * 4) = make_uint4(w[0], w[1], w[2], w[3]);
            }
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                int row, col;
                place(j, row, col);
                const uint4 v = *reinterpret_cast<const uint4 *>(slab + row * S::PITCH + (col - wc * 16 * NE) * 4);
                const int ml = wr * 16 * MI + 16 * i + row;
                if (m0 + ml < n_rows) ChunkOut<Store>(store, col, E).put(v, ext[READS ? i & 1 : 0][j], side.gate(ml), side.dest(ml));
            }
        }
    };
    if (store.accumulate) emit(std::true_type{});
    else emit(std::false_type{});
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

template <int NE, int MI>
int launch(const MlpArgs &a, hipStream_t st) {
    typedef ShiftStore<kEpiScatterI32> Store;
    const long blocks = (a.sel.max_rows + 32 * MI - 1) / (32 * MI);
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "sa_shift_mlp: too many rows for one launch");
    const dim3 grid((unsigned)blocks), block(kMlpWaves * 64);
    if (a.norm && a.norm->wo)
        shift_mlp_kernel<NE, MI, kProject, Store><<<grid, block, 0, st>>>(a.x, *a.norm, a.sel, a.hid, a.w1, a.w2, a.lut, a.rq, a.store);
    else if (a.norm)
        shift_mlp_kernel<NE, MI, kNorm, Store><<<grid, block, 0, st>>>(nullptr, *a.norm, a.sel, a.hid, a.w1, a.w2, a.lut, a.rq, a.store);
    else
        shift_mlp_kernel<NE, MI, kCodes, Store><<<grid, block, 0, st>>>(a.x, NormRows{}, a.sel, a.hid, a.w1, a.w2, a.lut, a.rq, a.store);
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
int sa::launch_shift_mlp(const int8_t *x, const NormRows *norm, const RowSel &sel, int E, int hid, const int8_t *w1_planes,
                         const int8_t *w2_planes, const int8_t *lut, float requant_scale, const Epilogue &out, hipStream_t st) {
    SA_REQUIRE(!norm || (!sel.rows && !out.gate), SA_ERR_INVALID, "sa_shift_mlp: rows to normalise are all rows, ungated");
    const MlpArgs a{x, norm, sel, hid, w1_planes, w2_planes, lut, requant_scale_finite(requant_scale), ShiftStore<kEpiScatterI32>(out)};
    const long m_est = sel.counts ? (sel.max_rows + 1) / 2 : sel.max_rows;
    auto rounds = [&](long rows) { return ((m_est + rows - 1) / rows + 255) / 256; };
    const bool tall = 29 * rounds(128) < 20 * rounds(64);
    switch (E) {
        case 64: return launch<1, 2>(a, st);
        case 128: return tall ? launch<2, 4>(a, st) : launch<2, 2>(a, st);
        case 192: return tall ? launch<3, 4>(a, st) : launch<3, 2>(a, st);
        case 256: return tall ? launch<4, 4>(a, st) : launch<4, 2>(a, st);
    }
    return fail(SA_ERR_UNSUPPORTED, "sa_shift_mlp: width %d in one launch", E);
}
