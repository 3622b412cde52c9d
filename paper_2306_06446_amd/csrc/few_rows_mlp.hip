// The MLP half of a layer, or the MLP of a block, for few rows of E = 64 .. 256 in one launch:
//     x' = x + Wo . codes (layer),  e = expert of LayerNorm(x') . wg + bg,  y = x' + gate * E_e(LayerNorm(x'))
// With few rows the launches of this chain are bound by their starts and by one round trip of loads each, and by waiting for one another: output
// projection with its LayerNorm 5.9, routing 3.4, first and second layers of the experts 5.5 + 5.8 us of the 37 that a DeiT-Tiny layer of one
// image took.  Here a workgroup has 16 rows, one expert and a quarter of its hidden columns.  It makes the rows and their LayerNorm itself, as
// its seven neighbours do (73 KB of Wo at E = 192, where its share of the expert's weights is 147), takes the decision from the row itself, and
// leaves partial sums of the output columns for those rows that are its expert's; of the four workgroups that have the same rows and expert the
// last one to get there adds the four.  Nobody waits for anybody.  One launch of 9.5 us: the layer 36.8 -> 25.7; of a block, whose routing rides in
// the hash's launch, the two layers 10.7 -> 7.
//
// A wavefront has 16 columns of everything.  Its weights come through a ring of its own, in pieces of 128 bytes of 16 rows, one behind the
// other over all three products: no barrier before a piece is read or its place is taken, and the next product's weights are on their way
// while the LayerNorm, the table or the GELU keep the wavefront.  What bounds a workgroup is its own chain, 8.1 us of it by its clock (197 x 192,
// two experts): first loads 0.9, Wo 1.0, LayerNorm 1.3, first layer 1.1 to 1.5, second 0.6, the partial sums' way to memory 0.7, the ticket
// 0.4, the way back and out 1.5.  32 columns to a wavefront and 32 rows took 13 us, 4.4 of them for a LayerNorm of 64 lanes to a row.
//
// Results are those of the launches it replaces, bit for bit where these take the tiles of gemm_slice.h: the row's sums are taken as in
// layernorm.hip, the Mult expert's as those tiles do, which split a contraction between four wavefronts 16 columns at a time: hence its hidden
// columns 64 i + 16 s .. + 15 are workgroup s's, whose partial sums are added in that order.
#include "common.h"
#include "gemm_common.h"
#include "gemm_mfma.h"
#include "gemm_stores.h"
#include "layernorm.h"

namespace {

using namespace sa;

typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef float v4f_t __attribute__((ext_vector_type(4)));

constexpr int kSlices = 4, kPiece = 2048;                    // piece: 128 bytes of 16 rows of weights

// MI: 16-row tiles of a workgroup
template <int NE, int MI>
struct FewRowsShape {
    static constexpr int E = 64 * NE, WAVES = 4 * NE, ROWS = 16 * MI;
    static constexpr int RING = NE * MI >= 8 || NE == 3 ? 2 : 3;        // pieces on their way to a wavefront
    static constexpr int MAX_HID = (NE * MI > 8 || NE == 3 ? 4 : 8) * E;
    // LDS: rings, rows as fp32, rows as operands (codes or fp16), hidden rows, parameters, table
    static constexpr int R = WAVES * RING * kPiece, X = R + ROWS * E * 4, H = X + ROWS * 2 * E;
    static constexpr int PARAMS = H + ROWS * (MAX_HID / 2 + 16);         // gamma, beta, router
    static constexpr int TABLE = PARAMS + 16 * E, LOGITS = TABLE + 256, FLAG = LOGITS + ROWS * 8 + 256, LDS_BYTES = FLAG + 16;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
};

struct FewRows {
    const int8_t *codes;             // of the attention's output (layer), of the MLP's rows (block)
    const _Float16 *half;            // block: the MLP's rows
    NormRows norm;                   // layer
    const float *wg, *bg;            // layer: router
    const float *logits;             // block
    long T;
    int hid;
    const int8_t *w1, *w2, *lut;
    const _Float16 *mw1, *mw2;
    float rq, out_scale;
    float *y;
    uint32_t *partials, *tickets;    // [tiles][kSlices][16 MI * E], [tiles][2]
};

// Physical 16-byte chunk of chunk c of LDS row r, rows of CPR chunks one behind the other: 16 consecutive rows hit 16 bank groups.
template <int CPR>
__device__ inline int spread(int r, int c) {
    if (CPR % 16 == 0) return c ^ (r & 15);
    if (CPR % 8 == 0) return c ^ ((r >> 1) & 7);
    return (c & ~3) | ((c & 3) ^ ((r >> 2) & 3));
}

// Memory that other workgroups of the launch write or read, on any XCD: past the L2s.
__device__ inline void put_shared(uint32_t *at, const uint4 &v) {
    uint64_t *p = reinterpret_cast<uint64_t *>(at);
    __hip_atomic_store(p, v.x | ((uint64_t)v.y << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p + 1, v.z | ((uint64_t)v.w << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint64_t get_shared(const uint32_t *at) {
    return __hip_atomic_load(reinterpret_cast<const uint64_t *>(at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline v4i_t mma16(const uint4 &a, const uint4 &b, v4i_t c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i_t, a), __builtin_bit_cast(v4i_t, b), c, 0, 0, 0);
}
__device__ inline v4f_t mma16(const uint4 &a, const uint4 &b, v4f_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h_t, a), __builtin_bit_cast(v8h_t, b), c, 0, 0, 0);
}

// SHIFT: the Shift expert (expert 1, or the only one); else the Mult expert.  LAYER: the rows are made and normalised here.
template <int NE, int MI, bool LAYER, bool MOE, bool SHIFT>
__device__ __forceinline__ void few_rows_tile(const FewRows &a, long tile, int slice, uint8_t *lds) {
    using S = FewRowsShape<NE, MI>;
    constexpr int E = S::E, WAVES = S::WAVES, kRows = S::ROWS, kRing = S::RING;
    typedef typename std::conditional<SHIFT, v4i_t, v4f_t>::type Acc;
    const int tid = threadIdx.x, lane = tid & 63, fr = lane & 15, fg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    const long m0 = tile * kRows, last = a.T - 1;
    const int hid = a.hid, mine = hid / kSlices;             // hidden columns of this workgroup
    const int tiles1 = mine / E, pieces2 = mine / 64;        // of a wavefront: column tiles of the first layer, pieces of the second's weights
    constexpr int PRE = LAYER ? NE : 0;
    const float bg0 = LAYER && MOE ? a.bg[0] : 0.0f, bg1 = LAYER && MOE ? a.bg[1] : 0.0f;
    const int pieces = PRE + tiles1 * NE + pieces2;

    // Piece p of this wavefront's weights: Wo's (of a row, the two planes are one behind the other), then the first layer's, 16 hidden columns
    // at a time, then the second's.  Load i of its two takes rows 8 i + lane / 8; what differs between the lanes is an offset for either, and
    // for planes whose seam lies inside a piece which side of it a chunk is on.
    const int b0 = spread<8>(lane / 8, lane % 8) * 16;       // byte of a piece's row (i = 1: ^ 64)
    uint32_t of_wo[2], of_w1[2], of_w2[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t r = 8 * i + lane / 8, b = b0 ^ (64 * i);
        of_wo[i] = r * E + b;
        of_w1[i] = r * (SHIFT ? E : 2 * E) + b;
        of_w2[i] = SHIFT ? r * hid + b : 2 * r * hid + b / 32 * 128 + b % 32;
    }
    // the Mult expert's hidden columns: 16 of every 64
    const int8_t *wo = a.norm.wo + (size_t)(16 * wave) * E;
    const int8_t *w1 = SHIFT ? a.w1 + (size_t)(slice * mine + 16 * wave) * E : reinterpret_cast<const int8_t *>(a.mw1) + (size_t)(64 * wave + 16 * slice) * (2 * E);
    const int8_t *w2 = SHIFT ? a.w2 + (size_t)(16 * wave) * hid + slice * mine : reinterpret_cast<const int8_t *>(a.mw2) + (size_t)(16 * wave) * (2 * hid) + 32 * slice;
    const uint32_t ring = wave * (kRing * kPiece);
    // base: of the piece; seam: byte of the piece behind which the second plane lies `jump` further on
    auto issue_piece = [&](const int8_t *base, const uint32_t (&of)[2], bool planes, int seam, uint32_t jump, int slot) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t off = of[i];
            if (planes) off += (b0 ^ (64 * i)) >= seam ? jump : 0u;
            direct_load_16(base, off, lds_base + ring + slot * kPiece + i * 1024);
        }
    };
    auto issue = [&](int p, int slot) {
        if (LAYER && p < PRE) return issue_piece(wo + 128 * p, of_wo, true, E - 128 * p, E * E - E, slot);
        p -= PRE;
        if (p < tiles1 * NE) {
            const int t = p / NE, c = p - t * NE;
            if (SHIFT) issue_piece(w1 + (size_t)(t * WAVES * 16) * E + 128 * c, of_w1, true, E - 128 * c, (uint32_t)(hid * E - E), slot);
            else issue_piece(w1 + (size_t)(t * WAVES * 64) * (2 * E) + 128 * c, of_w1, false, 0, 0, slot);
            return;
        }
        p -= tiles1 * NE;
        if (SHIFT) issue_piece(w2 + 128 * p, of_w2, true, mine - 128 * p, (uint32_t)(E * hid - mine), slot);
        else issue_piece(w2 + 512 * p, of_w2, false, 0, 0, slot);
    };

    // ---- what all wavefronts read: the attention's codes and the residual (layer) or the rows; parameters, table
    auto load_rows = [&](const void *from, auto cpr_c, uint32_t to) {
        constexpr int CPR = decltype(cpr_c)::value, KIB = kRows * CPR / 64;
        for (int i = wave; i < KIB; i += WAVES) {
            const int c = i * 64 + lane, r = c / CPR;
            direct_load_16(static_cast<const uint8_t *>(from) + (size_t)min(m0 + r, last) * (16 * CPR) + spread<CPR>(r, c % CPR) * 16,
                           lds_base + to + i * 1024);
        }
    };
    if constexpr (LAYER) {
        load_rows(a.codes, std::integral_constant<int, 4 * NE>{}, S::X);
        load_rows(a.norm.residual, std::integral_constant<int, 16 * NE>{}, S::R);
        if (wave < (MOE ? 4 : 2) * NE) {                     // 256 bytes each: gamma, beta, the router's two columns
            const float *from = wave < NE ? a.norm.gamma + 64 * wave : wave < 2 * NE ? a.norm.beta + 64 * (wave - NE) : a.wg + 64 * (wave - 2 * NE);
            direct_load_4(from + lane, lds_base + S::PARAMS + wave * 256);
        }
    } else {
        if constexpr (SHIFT) load_rows(a.codes, std::integral_constant<int, 4 * NE>{}, S::X);
        else load_rows(a.half, std::integral_constant<int, 8 * NE>{}, S::X);
        if constexpr (MOE)
            if (wave < (kRows + 31) / 32) direct_load_4(a.logits + min(2 * (m0 + 32 * wave) + lane, 2 * last + 1), lds_base + S::LOGITS + wave * 256);
    }
    if constexpr (SHIFT)
        if (wave == WAVES - 1) direct_load_4(a.lut + lane * 4, lds_base + S::TABLE);
#pragma unroll
    for (int p = 0; p < kRing; ++p)
        if (p < pieces) issue(p, p);

    int piece = 0, slot = 0;                                 // the next one to be multiplied, its place in the ring
    // until n pieces from the next one on are there
    auto arrive = [&](int n) {
        const int later = pieces - n - piece;
        if (kRing - n >= 2 && later >= 2) wait_loads_in_flight<4>();
        else if (kRing - n >= 1 && later >= 1) wait_loads_in_flight<2>();
        else wait_loads_in_flight<0>();
    };
    static_assert(kRing == 2 || kRing == 3, "arrive");
    auto chunk = [&](int s, int c) { return *reinterpret_cast<const uint4 *>(lds + ring + s * kPiece + fr * 128 + spread<8>(fr, c) * 16); };
    auto next = [](int s) { return s == kRing - 1 ? 0 : s + 1; };
    auto leave = [&]() {                                     // its operands are in registers: its place for the piece kRing further on
        if (piece + kRing < pieces) issue(piece + kRing, slot);
        ++piece;
        slot = next(slot);
    };
    arrive(1);
    __syncthreads();

    // Products are computed transposed (weights down, rows across): register r of a lane is column 4 fg + r of the wavefront's 16, of row
    // lane % 16 of a tile.
    auto row_chunk = [&](int r, int c) { return reinterpret_cast<float4 *>(lds + S::R + (r * 16 * NE + spread<16 * NE>(r, c)) * 16); };
    if constexpr (LAYER) {
        v4i_t acc[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[i] = v4i_t{0, 0, 0, 0};
#pragma unroll
        for (int c = 0; c < NE; ++c) {
            arrive(1);
            const uint4 b[2] = {chunk(slot, fg), chunk(slot, 4 + fg)};
            uint4 rows[2][MI];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    rows[q][i] = *reinterpret_cast<const uint4 *>(lds + S::X + (16 * i + fr) * E + spread<4 * NE>(fr, (128 * c + 64 * q) % E / 16 + fg) * 16);
            wait_lds_reads();
            leave();
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < MI; ++i) acc[i] = mma16(b[q], rows[q][i], acc[i]);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            float4 *at = row_chunk(16 * i + fr, 4 * wave + fg);
            const float4 res = *at;
            *at = make_float4(__builtin_fmaf((float)acc[i][0], a.norm.scale, res.x), __builtin_fmaf((float)acc[i][1], a.norm.scale, res.y),
                              __builtin_fmaf((float)acc[i][2], a.norm.scale, res.z), __builtin_fmaf((float)acc[i][3], a.norm.scale, res.w));
        }
        __syncthreads();                                     // the rows are complete, the codes have been read

        // ---- LayerNorm: 16 lanes a row, four rows of a wavefront (a row on each of its lanes' own took twice the instructions).  The sums are
        //      added as layernorm.hip does with 16 NE lanes a row: the most distant first.
        const float *params = reinterpret_cast<const float *>(lds + S::PARAMS);
        auto row_sum = [](const float (&v)[NE]) {
            if constexpr (NE == 1) return group_sum<16>(v[0]);
            else if constexpr (NE == 2) return group_sum<16>(v[0] + v[1]);
            else return group_sum<16>((v[0] + v[2]) + (v[1] + (NE == 4 ? v[NE - 1] : 0.0f)));
        };
        for (int r = 4 * wave + fg; r < kRows; r += 4 * WAVES) {             // (a whole wavefront's rows end together)
            float4 x[NE];
            float sum[NE];
#pragma unroll
            for (int c = 0; c < NE; ++c) {
                x[c] = *row_chunk(r, 16 * c + fr);
                sum[c] = (x[c].x + x[c].y) + (x[c].z + x[c].w);
            }
            const float mean = row_sum(sum) / (float)E;
#pragma unroll
            for (int c = 0; c < NE; ++c) {
                const float d0 = x[c].x - mean, d1 = x[c].y - mean, d2 = x[c].z - mean, d3 = x[c].w - mean;
                sum[c] = (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
            }
            const float rstd = 1.0f / __builtin_sqrtf(row_sum(sum) / (float)E + a.norm.eps);
            float part[2][NE];
#pragma unroll
            for (int c = 0; c < NE; ++c) {
                const int j = 64 * c + 4 * fr;
                float y[4];
                normalise(x[c], mean, rstd, *reinterpret_cast<const float4 *>(params + j), *reinterpret_cast<const float4 *>(params + E + j), y);
                if constexpr (SHIFT)
                    *reinterpret_cast<uint32_t *>(lds + S::X + r * E + spread<4 * NE>(r, 4 * c + fr / 4) * 16 + fr % 4 * 4) = codes_of(y, a.norm.inv_scale);
                else
                    *reinterpret_cast<v4h *>(lds + S::X + r * 2 * E + spread<8 * NE>(r, 8 * c + fr / 2) * 16 + fr % 2 * 8) =
                        v4h{(_Float16)y[0], (_Float16)y[1], (_Float16)y[2], (_Float16)y[3]};
                if constexpr (MOE) {
                    const float4 w0 = *reinterpret_cast<const float4 *>(params + 2 * E + 2 * j), w1 = *reinterpret_cast<const float4 *>(params + 2 * E + 2 * j + 4);
                    part[0][c] = __builtin_fmaf(y[3], w1.z, __builtin_fmaf(y[2], w1.x, __builtin_fmaf(y[1], w0.z, __builtin_fmaf(y[0], w0.x, 0.0f))));
                    part[1][c] = __builtin_fmaf(y[3], w1.w, __builtin_fmaf(y[2], w1.y, __builtin_fmaf(y[1], w0.w, __builtin_fmaf(y[0], w0.y, 0.0f))));
                }
            }
            if constexpr (MOE) {
                const float l0 = row_sum(part[0]) + bg0, l1 = row_sum(part[1]) + bg1;
                if (fr == 0) *reinterpret_cast<float2 *>(lds + S::LOGITS + 8 * r) = make_float2(l0, l1);
            }
        }
        __syncthreads();
    }

    // ---- whose rows 16 i + lane % 16 are
    bool own[MI], any = false;
    auto logits_of = [&](int i) { return reinterpret_cast<const float2 *>(lds + S::LOGITS)[16 * i + fr]; };
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        own[i] = m0 + 16 * i + fr <= last;
        if constexpr (MOE) {
            const float2 lg = logits_of(i);
            own[i] = own[i] && (lg.y > lg.x) == SHIFT;
        }
        any = any || own[i];
    }
    if (MOE && __ballot(any) == 0) {                         // in all wavefronts of the four workgroups
        wait_loads_in_flight<0>();                           // (nothing may arrive in LDS that is another workgroup's by then)
        return;
    }

    // ---- first layer: 16 hidden columns of a wavefront at a time.  The Mult expert's sums are those of the tiles of gemm_slice.h, which split
    //      this contraction in two (rows of 512 bytes and more: in four), 16 of it at a time: a product here takes two such pieces of
    //      one share one behind the other, which is what two products of 16 would do (the same bits).
    constexpr int XB = SHIFT ? E : 2 * E;                    // bytes of a row
    constexpr int PARTS = SHIFT ? 1 : NE == 4 ? 4 : 2;
    auto x_chunk = [&](int i, int c) { return *reinterpret_cast<const uint4 *>(lds + S::X + (16 * i + fr) * XB + spread<XB / 16>(fr, c) * 16); };
    const int pitch = (SHIFT ? mine : 2 * mine) + 16;
    for (int t = 0; t < tiles1; ++t) {
        Acc acc[MI][PARTS];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int p = 0; p < PARTS; ++p) acc[i][p] = Acc{0, 0, 0, 0};
        if constexpr (PARTS < 4) {
#pragma unroll
            for (int c = 0; c < NE; ++c) {
                const int at = SHIFT ? fg : 4 * (fg / 2) + fg % 2, step = SHIFT ? 4 : 2;
                arrive(1);
                const uint4 b[2] = {chunk(slot, at), chunk(slot, at + step)};
                uint4 rows[2][MI];
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int i = 0; i < MI; ++i) rows[q][i] = x_chunk(i, SHIFT ? (128 * c + 64 * q) % E / 16 + fg : 8 * c + at + step * q);
                wait_lds_reads();
                leave();
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int i = 0; i < MI; ++i) acc[i][q % PARTS] = mma16(b[q], rows[q][i], acc[i][q % PARTS]);
            }
        } else {
#pragma unroll
            for (int c = 0; c < NE; c += 2) {
                arrive(2);
                uint4 b[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) b[q] = chunk(fg < 2 ? slot : next(slot), 2 * q + fg % 2);
                wait_lds_reads();
                leave();
                leave();
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < MI; ++i) acc[i][q % PARTS] = mma16(b[q], x_chunk(i, 8 * (c + fg / 2) + 2 * q + fg % 2), acc[i][q % PARTS]);
            }
        }
        const int col = 16 * (wave + t * WAVES) + 4 * fg;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            uint8_t *to = lds + S::H + (16 * i + fr) * pitch;
            if constexpr (SHIFT) {
                uint32_t v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = lds[S::TABLE + requant_index(acc[i][0][e], a.rq)];
                *reinterpret_cast<uint32_t *>(to + col) = (v[0] | (v[1] << 8)) | ((v[2] | (v[3] << 8)) << 16);
            } else {
                v4h h;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float sum = acc[i][0][e];
#pragma unroll
                    for (int p = 1; p < PARTS; ++p) sum += acc[i][p][e];
                    h[e] = (_Float16)gelu_erf(sum);
                }
                *reinterpret_cast<v4h *>(to + 2 * col) = h;
            }
        }
    }
    __syncthreads();

    // ---- second layer: this workgroup's share of the contraction
    Acc acc[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) acc[i] = Acc{0, 0, 0, 0};
    for (int c = 0; c < pieces2; ++c) {
        arrive(1);
        const uint4 b[2] = {chunk(slot, fg), chunk(slot, 4 + fg)};
        uint4 rows[2][MI];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            int k = 128 * c + 64 * q;                        // byte of a hidden row (the second plane takes them once more)
            if (SHIFT && k >= mine) k -= mine;
#pragma unroll
            for (int i = 0; i < MI; ++i) rows[q][i] = *reinterpret_cast<const uint4 *>(lds + S::H + (16 * i + fr) * pitch + k + 16 * fg);
        }
        wait_lds_reads();
        leave();
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < MI; ++i) acc[i] = mma16(b[q], rows[q][i], acc[i]);
    }

    // ---- partial sums, of this expert's rows only (the other's have the same place)
    constexpr size_t SLICE = kRows * E;
    uint32_t *part = a.partials + (size_t)tile * kSlices * SLICE + wave * (256 * MI) + lane * 4;
    auto bits = [](auto v) { return __builtin_bit_cast(uint32_t, v); };
#pragma unroll
    for (int i = 0; i < MI; ++i)
        if (own[i]) put_shared(part + slice * SLICE + 256 * i, make_uint4(bits(acc[i][0]), bits(acc[i][1]), bits(acc[i][2]), bits(acc[i][3])));
    wait_loads_in_flight<0>();                               // they are in memory
    __syncthreads();                                         // all wavefronts' are
    uint32_t *flag = reinterpret_cast<uint32_t *>(lds + S::FLAG);
    if (tid == 0) *flag = __hip_atomic_fetch_add(a.tickets + 2 * tile + (SHIFT ? 1 : 0), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*flag != kSlices - 1) return;
    uint64_t got[MI][kSlices][2];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int s = 0; s < kSlices; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h) got[i][s][h] = own[i] ? get_shared(part + s * SLICE + 256 * i + 2 * h) : 0;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            auto word = [&](int s) { return (uint32_t)(got[i][s][e / 2] >> (32 * (e % 2))); };
            if constexpr (SHIFT) {
                uint32_t sum = 0;
#pragma unroll
                for (int s = 0; s < kSlices; ++s) sum += word(s);
                v[e] = a.out_scale * (float)(int32_t)sum;
            } else {
                v[e] = __builtin_bit_cast(float, word(0));
#pragma unroll
                for (int s = 1; s < kSlices; ++s) v[e] += __builtin_bit_cast(float, word(s));
            }
        }
        float gate = 1.0f;                                   // as route_scatter_block takes it
        if constexpr (MOE) {
            const float2 lg = logits_of(i);
            const float top = SHIFT ? lg.y : lg.x;
            gate = 1.0f / (__expf(lg.x - top) + __expf(lg.y - top));
        }
        if constexpr (LAYER) {
            const float4 old = *row_chunk(16 * i + fr, 4 * wave + fg);
            v[0] = __builtin_fmaf(gate, v[0], old.x);
            v[1] = __builtin_fmaf(gate, v[1], old.y);
            v[2] = __builtin_fmaf(gate, v[2], old.z);
            v[3] = __builtin_fmaf(gate, v[3], old.w);
        } else if constexpr (MOE) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= gate;
        }
        if (own[i]) *reinterpret_cast<float4 *>(a.y + (size_t)(m0 + 16 * i + fr) * E + 16 * wave + 4 * fg) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

// Workgroup b: share b % 4 of expert b / 4 % 2 for rows b / 8 ..: workgroups are handed to the XCDs in turn, so each L2 fetches one share.
template <int NE, int MI, bool LAYER, bool MOE>
__global__ __launch_bounds__(NE * 256) void few_rows_kernel(FewRows a) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[FewRowsShape<NE, MI>::LDS_BYTES];
    const int slice = blockIdx.x % kSlices, rest = blockIdx.x / kSlices;
    if constexpr (MOE) {
        if (rest % 2 == 0) few_rows_tile<NE, MI, LAYER, true, false>(a, rest / 2, slice, lds);
        else few_rows_tile<NE, MI, LAYER, true, true>(a, rest / 2, slice, lds);
    } else {
        few_rows_tile<NE, MI, LAYER, false, true>(a, rest, slice, lds);
    }
}

template <int NE, int MI>
int launch(const FewRows &a, bool layer, bool moe, hipStream_t st) {
    const long tiles = (a.T + 16 * MI - 1) / (16 * MI);
    const dim3 grid((unsigned)(tiles * kSlices * (moe ? 2 : 1))), block(NE * 256);
    if (layer && moe) few_rows_kernel<NE, MI, true, true><<<grid, block, 0, st>>>(a);
    else if (layer) few_rows_kernel<NE, MI, true, false><<<grid, block, 0, st>>>(a);
    else if (moe) few_rows_kernel<NE, MI, false, true><<<grid, block, 0, st>>>(a);
    else few_rows_kernel<NE, MI, false, false><<<grid, block, 0, st>>>(a);
    return check_launch("MLP of few rows");
}

template <int NE>
int launch_width(const FewRows &a, int mi, bool layer, bool moe, hipStream_t st) {
    if (mi == 1) return launch<NE, 1>(a, layer, moe, st);
    if constexpr (NE >= 3) {                                 // layers only (plan_few_rows)
        const dim3 grid((unsigned)((a.T + 16 * mi - 1) / (16 * mi) * kSlices * (moe ? 2 : 1))), block(NE * 256);
        if (layer && mi == 2) {
            if (moe) few_rows_kernel<NE, 2, true, true><<<grid, block, 0, st>>>(a);
            else few_rows_kernel<NE, 2, true, false><<<grid, block, 0, st>>>(a);
            return check_launch("MLP of few rows");
        }
        if constexpr (NE == 3) {
            if (layer && moe && mi == 4) {
                few_rows_kernel<3, 4, true, true><<<grid, block, 0, st>>>(a);
                return check_launch("MLP of few rows");
            }
        }
    }
    return fail(SA_ERR_UNSUPPORTED, "MLP of few rows: %d tiles to a workgroup", mi);
}

}  // namespace

// Where it is the faster way: up to kMost workgroups of 16 rows, of which a CU has LDS for four at E = 64, two at 128 and 192, one at 256.
// Where it replaces many launches (layers of two experts) that is more than one round of them, else less than one.  Whole layers and blocks of
// 64-bit codes and linear attention, hid = 4 E (E = 64: 8 E), launches of their own against this one, us:
//   layer, two experts  E =  64:   784 rows 31.5, 21.8; 3136 35.0, 29.2; 6272 41.7, 39.6; 9408 47.0, 47.1
//                       E = 128:   200 rows 31.3, 20.4; 1600 34.7, 28.8; 2400 36.3, 33.9; 3200 39.9, 42.0
//                       E = 192:   197 rows 36.8, 25.7;  394 37.6, 26.6
//                       E = 256:    49 rows 34.7, 24.0;  392 36.6, 26.1
//   layer, Shift        E =  64:   784 rows 22.1, 20.6; 1568 22.1, 21.4; 3136 22.6, 22.9
//                       E = 128:   200 rows 24.6, 19.7; 1600 25.4, 22.5; 2400 25.8, 27.0
//                       E = 192:   197 rows 29.3, 25.0;  985 30.7, 26.7
//                       E = 256:    49 rows 28.2, 23.8;  980 31.2, 26.1
//   block, two experts  E =  64:   784 rows 23.7, 20.6; 1568 24.7, 23.0; 2352 25.6, 26.3
//                       E = 128:   200 rows 22.4, 18.4;  800 22.9, 21.0; 1600 24.1, 26.0
//                       E = 192:   197 rows 23.5, 19.9;  394 23.8, 21.0;  591 24.0, 25.5
//                       E = 256:    49 rows 21.0, 18.1;  392 21.8, 20.9;  490 21.9, 22.3
//   block, Shift        E =  64:   784 rows 20.3, 19.6; 1568 20.5, 20.1; 2352 20.9, 21.2
//                       E = 128:   200 rows 20.7, 17.9; 1600 21.6, 20.4; 2400 21.8, 23.8
//                       E = 192:   197 rows 20.3, 19.4;  985 21.4, 20.8; 1182 22.5, 24.0
//                       E = 256:    49 rows 17.9, 18.1;  784 20.4, 20.0: not taken
// hid = 8 E (E = 64: 4 E), of which a Shift block of E = 64 gains nothing and a workgroup of E = 256 has twice the chain:
//   layer, two experts  E =  64:   735 rows 29.5, 17.7; 6174 34.2, 31.2         E = 128: 294 rows 32.2, 19.6; 1274 34.3, 29.9; 2450 37.9, 38.1
//                       E = 256:    98 rows 39.4, 28.4;  490 41.0, 35.6; 980 44.5, 40.3
//   layer, Shift        E =  64:   784 rows 17.4, 16.6; 1519 17.5, 16.9         E = 128: 882 rows 25.7, 20.0; 1715 27.8, 21.9
//                       E = 256:   245 rows 32.3, 27.1;  980 35.2, 28.4; 1960 44.8, 39.8
//   block, two experts  E =  64:   784 rows 21.1, 17.1; 1519 21.0, 18.3         E = 128: 490 rows 22.6, 18.9;  980 23.2, 22.4
//                       E = 256:    98 rows 23.6, 22.2;  147 23.9, 23.7;  392 24.9, 26.4
//   block, Shift        E =  64:   784 rows 14.3, 14.5; 1519 14.5, 15.5: not taken      E = 128: 784 rows 19.9, 17.9; 1519 21.1, 19.7
// The sign hash, codes of 128 and 256 bits, Hamming attention and packed weights: over the same rows between 1 % slower (at their ends) and 1.8
// times as fast.
// More rows of wide layers, whose chain is the longest, with 32 or 64 of them to a workgroup as long as those are one round:
//   two experts  E = 192, 32 rows:  591 rows 38.0, 29.4; 985 39.6, 31.8; 64 rows: 1182 41.1, 36.9; 1970 45.0, 42.9
//                E = 256, 32 rows:  588 rows 38.1, 30.9; 980 40.2, 32.9; 1176 (a second round) 42.0, 42.4
//   Shift        E = 192, 32 rows: 1182 rows 31.9, 29.0; 1970 36.2, 34.3     E = 256, 32 rows: 1176 32.6, 29.6; 1568 38.3, 35.8
sa::FewRowsPlan sa::plan_few_rows(long T, int E, int hid, bool moe, bool layer) {
    FewRowsPlan p;
    if (T <= 0 || E <= 0 || E % 64 != 0 || E > 256 || hid % (4 * E) != 0 || hid > (E == 192 ? 4 : 8) * E) return p;
    const int ne = E / 64;
    // by hid: 4 E, 8 E (none of E = 192); by E
    static const int kMost[2][2][2][4] = {{{{0, 400, 256, 0}, {400, 400, 0, 0}}, {{800, 512, 256, 208}, {800, 512, 0, 56}}},                // block: Shift, two experts
                                          {{{400, 448, 256, 256}, {400, 448, 0, 256}}, {{3200, 1280, 256, 256}, {3200, 1152, 0, 256}}}};    // layer
    auto groups = [&](int mi) { return (T + 16 * mi - 1) / (16 * mi) * kSlices * (moe ? 2 : 1); };
    if (groups(1) > kMost[layer][moe][hid > 4 * E][ne - 1]) {
        if (!layer || ne < 3) return p;
        if (groups(2) <= 256) p.mi = 2;
        else if (ne == 3 && moe && groups(4) <= 256) p.mi = 4;
        else return p;
    }
    const long tiles = (T + 16 * p.mi - 1) / (16 * p.mi);
    p.ticket_bytes = (size_t)tiles * 2 * 4;
    p.bytes = (p.ticket_bytes + 255) / 256 * 256 + (size_t)tiles * kSlices * 16 * p.mi * E * 4;
    return p;
}

int sa::launch_few_rows(const FewRowsMlp &m, const FewRowsPlan &p, hipStream_t st) {
    uint8_t *ws = static_cast<uint8_t *>(m.workspace);
    const size_t tickets = (p.ticket_bytes + 255) / 256 * 256;
    const FewRows a{m.codes, static_cast<const _Float16 *>(m.half), m.norm ? *m.norm : NormRows(), m.wg, m.bg, m.logits, m.T, m.hid, m.w1, m.w2, m.lut,
                    static_cast<const _Float16 *>(m.mw1), static_cast<const _Float16 *>(m.mw2), requant_scale_finite(m.requant_scale), m.out_scale, m.y,
                    reinterpret_cast<uint32_t *>(ws + tickets), reinterpret_cast<uint32_t *>(ws)};
    const bool layer = m.norm != nullptr, moe = m.mw1 != nullptr;
    switch (m.E) {
        case 64: return launch_width<1>(a, p.mi, layer, moe, st);
        case 128: return launch_width<2>(a, p.mi, layer, moe, st);
        case 192: return launch_width<3>(a, p.mi, layer, moe, st);
        case 256: return launch_width<4>(a, p.mi, layer, moe, st);
    }
    return fail(SA_ERR_UNSUPPORTED, "MLP of few rows of width %d", m.E);
}
