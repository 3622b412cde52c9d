// Tiled "NT" matrix-core GEMM shared by the Shift expert (int8 x two int8 weight planes,
// int32 accumulate) and the Mult expert (fp16 x fp16, fp32 accumulate):
//     C[m, n] = sum_p sum_k A[m, k] * B_p[n, k]
//
// Workgroup tile BM x BN, four wavefronts in a 2 x 2 grid, each owning (BM/2) x (BN/2) as
// 32x32 MFMA tiles.  K advances SB bytes (64 or 128) per stage through a ring of NS (2 to 4) LDS
// stage buffers that is filled by direct global->LDS loads (no register staging): while stage s
// is multiplied out of one buffer, the loads of the following stages are in flight into the
// others; one barrier per stage; the LDS fragment reads run one 32-byte step ahead of the MFMAs
// that consume them, and the loads of a stage are spread between the MFMAs of LS steps.  A direct
// load writes 1 KiB of consecutive LDS per wavefront instruction, so LDS rows cannot be padded;
// instead the 16-byte chunks of a row are XOR-swizzled with the row number (the lane chooses
// which global chunk it fetches), which makes the 16-byte fragment reads of any 16 consecutive
// rows hit 16 different bank groups.
//
// The loads are issued from inline assembly: the kernel orders them by hand (one vmcnt wait and
// one barrier per stage), and the compiler must not serialise the reads of the current buffer
// behind the loads in flight into the other ones.  The K loop is written out in five pieces
// (first stage, steady state, the stage after which no load is left to issue, the stages that
// only drain, the last stage) so that the steady state holds no branch around a load and no
// branch join in front of its MFMAs.
//
// Outputs leave through LDS, so that every lane stores 16 bytes of one row (a scattered destination row
// index and its gate are then fetched once per 16 bytes).
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.h"
#include "gemm_common.h"
#include "side_work.h"

namespace sa {

// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), unrolled at compile time.
template <int... I, class F>
__device__ inline void static_for_impl(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ inline void static_for(F &&f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));
typedef _Float16 v8h_t __attribute__((ext_vector_type(8)));
typedef float v16f_t __attribute__((ext_vector_type(16)));

struct I8Traits {
    typedef v16i_t Acc;
    static constexpr int kPlanes = 2;
    static constexpr int kElemBytes = 1;
    static constexpr bool kPacked = false;
    __device__ static inline Acc mma(const uint4 &a, const uint4 &b, Acc c) {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(v4i_t, a), __builtin_bit_cast(v4i_t, b), c,
                                                     0, 0, 0);
    }
};

// The same products on packed 4-bit weights: a stage of B is decoded into its two planes on the way into LDS.
struct I8PackedTraits : I8Traits {
    static constexpr bool kPacked = true;
};

struct F16Traits {
    typedef v16f_t Acc;
    static constexpr int kPlanes = 1;
    static constexpr int kElemBytes = 2;
    static constexpr bool kPacked = false;
    __device__ static inline Acc mma(const uint4 &a, const uint4 &b, Acc c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h_t, a), __builtin_bit_cast(v8h_t, b), c,
                                                      0, 0, 0);
    }
};

// What the kernel needs to know about its operands.
struct GemmArgs {
    const void *a;          // [rows, K] elements, row-major
    const void *b[2];       // planes, each [N, K] elements, row-major (kPacked: b[0] alone, [N, K / 2] bytes)
    RowSel sel;             // which rows of A / of the scattered output
    bool gather_a;          // A rows are sel.rows[m] (else compact m)
    int K, N;               // K: extent of the contraction, a whole number of 64-byte stages; row length of the B planes
    // How the tiles are shared out to the XCDs (see tile_of), set by the launcher with share_out.  Kernels start with this: made there
    // from col_groups, divisions one after the other came before every tile's first load (two experts in one launch: 576 instructions, now 130;
    // 12608 x 768 <- 768 as a Mult and a Shift expert 30.35 -> 30.14 us, 12608 x 1536 <- 384 and back 50.1 -> 49.6; 25000 x 768 <- 256 32.1 -> 32.7 and
    // 12608 x 768 <- 256, 70 %, 20.8 -> 20.4, by how a round's workgroups fall in step).
    int log_groups = 0, col_tiles = 0, cols_per_group = 1;
    FastDiv by_cols{1};
    void share_out(int BN, int col_groups) {
        for (log_groups = 0; 1 << log_groups < col_groups;) ++log_groups;
        col_tiles = (N + BN - 1) / BN;
        cols_per_group = (col_tiles + col_groups - 1) / col_groups;
        by_cols = FastDiv((uint32_t)cols_per_group);
    }
    // Workgroups are handed to the 8 XCDs round-robin by their linear id, and each XCD has its own 4 MiB L2.  The 8 XCDs form a (8 /
    // col_groups) x col_groups grid over the output (col_groups = 1, 2, 4 or 8): an XCD owns every (8 / col_groups)-th row tile and every
    // col_groups-th column tile, and walks them row tile by row tile.
    __device__ __forceinline__ void tile_of(int block, int &row_tile, int &col_tile) const {
        const int xcd = block & 7, slot = block >> 3, row = (int)by_cols((uint32_t)slot);
        row_tile = (row << (3 - log_groups)) + (xcd >> log_groups);
        col_tile = ((slot - row * cols_per_group) << log_groups) + (xcd & ((1 << log_groups) - 1));
    }
    // A rows may be shorter than K (int8 only, 64-byte stages): a_valid elements, a multiple of 16 bytes, at a row
    // pitch of a_ld elements; 0 = K.  The B planes must then hold zeros from a_valid on: the kernel multiplies
    // those zeros with bytes it re-reads from inside the row, so it never reads past a row's end.
    int a_ld = 0, a_valid = 0;
    // Tiles with BLOCKED take A in columns of 64 bytes, a_block bytes from one to the next, each holding its rows one behind
    // the other.
    size_t a_block = 0;
};

// Physical 16-byte chunk of logical chunk c in LDS row r, for rows of CPR chunks.
template <int CPR>
__device__ inline int swizzle(int r, int c) {
    return c ^ ((r / (16 / CPR)) & (CPR - 1));
}

// A Store type says how accumulators become output rows:
//   static constexpr int  kBytes      : bytes per output element (1, 2 or 4)
//   static constexpr int  kTableBytes : 0, or 256 for a byte table that is copied into LDS
//   static constexpr bool kScatter    : output row of tile row m is sel.rows[m] (else m)
//   uint32_t convert(acc, int n, const uint8_t *lds_table) const : the element's bits for column n
//   void *out : [rows, N] elements;  const void *table;  const float *gate : null, or a factor per
//       destination row that multiplies fp32 outputs (kScatter && kBytes == 4 only);  bool accumulate :
//       (same case) the product is added to what the destination holds, as fma(gate, value, old)
//   static constexpr bool kSignCodes  : tiles left of column code_cols leave as packed sign bits instead
//       (bit = acc >= 0, 64 columns = one word): uint64_t *codes[2] (column block 0 / 1 of width part_width,
//       laid out [batch, head, token, word]), int head_dim (64 or 128), tokens (per batch element), heads
//   static constexpr int  kHashBytes  : (kSignCodes only) 0, or the LDS that hash(acc, lds, m, n_rows, col, tid) takes, which makes code
//       words of those tiles' rows in place of their sign bits
//   static constexpr bool kLinear     : fp32 outputs leave as fma(value, scale, residual[m, n]) into
//       column blocks: float *parts[3], int part_width (a multiple of 4), const float *residual, float scale

// The 16-byte chunks at columns n .. n + 16 / kBytes - 1 of the output: where they go, and what they need from memory besides
// the product (the residual, or what the destination holds).  fetch() is apart from put() so that the reads of many chunks
// are in flight at once: read where it was used, each waited for the one before it (two, with a row index and its gate).
// Small shift linears 58.4 -> 54.4 us, 12608 x 768 tokens through a layer 362 -> 335, moe linear 32.7 -> 29.6.
template <class Store>
struct ChunkOut {
    static constexpr int ES = Store::kBytes;
    const Store &store;
    uint8_t *dst;              // the chunk in row 0 of the output
    const float *res = nullptr;
    size_t pitch, res_pitch;
    int live;                  // elements of the chunk inside a row
    bool whole_chunks;         // no chunk straddles a row's end

    __device__ __forceinline__ ChunkOut(const Store &s, int n, int N) : store(s), pitch((size_t)N * ES), res_pitch(N), live(N - n) {
        whole_chunks = pitch % 16 == 0;
        dst = static_cast<uint8_t *>(s.out) + (size_t)n * ES;
        if constexpr (ES < 4) {                    // hidden rows in columns of 64 bytes (GemmArgs::a_block)
            if (s.out_block) {
                dst = static_cast<uint8_t *>(s.out) + (size_t)(n * ES / 64) * s.out_block + n * ES % 64;
                pitch = 64;
            }
        }
        if constexpr (Store::kLinear) {            // whole chunks by construction: part_width and N are multiples of 4
            const int part = n / s.part_width;
            float *base = part == 0 ? s.parts[0] : part == 1 ? s.parts[1] : s.parts[2];
            dst = reinterpret_cast<uint8_t *>(base + (n - part * s.part_width));
            pitch = (size_t)s.part_width * ES;
            if (s.residual) res = s.residual + min(n, N - 4);
        }
    }
    static constexpr bool MAY_READ = ES == 4 && !Store::kSignCodes && (Store::kLinear || Store::kScatter);
    __device__ __forceinline__ bool reads() const {
        if constexpr (MAY_READ && Store::kLinear) return res != nullptr;
        else if constexpr (MAY_READ) return store.accumulate;
        return false;
    }
    __device__ __forceinline__ float4 fetch(long t) const {
        float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (Store::kLinear && !Store::kSignCodes) {
            if (res) return *reinterpret_cast<const float4 *>(res + t * res_pitch);
        } else if constexpr (Store::kScatter && ES == 4) {
            if (store.accumulate && live > 0) {
                const float *old = reinterpret_cast<const float *>(dst + t * pitch);
                if (whole_chunks) return *reinterpret_cast<const float4 *>(old);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < live) x[e] = old[e];
            }
        }
        return make_float4(x[0], x[1], x[2], x[3]);
    }
    // v: converted elements; x: what fetch() gave; gate: the factor of destination row t
    __device__ __forceinline__ void put(uint4 v, float4 x, float gate, long t) const {
        auto as_float = [](uint32_t b) { return __builtin_bit_cast(float, b); };
        auto as_bits = [](float f) { return __builtin_bit_cast(uint32_t, f); };
        if constexpr (Store::kLinear) {
            v = make_uint4(as_bits(__builtin_fmaf(as_float(v.x), store.scale, x.x)), as_bits(__builtin_fmaf(as_float(v.y), store.scale, x.y)),
                           as_bits(__builtin_fmaf(as_float(v.z), store.scale, x.z)), as_bits(__builtin_fmaf(as_float(v.w), store.scale, x.w)));
        } else if constexpr (Store::kScatter && ES == 4) {
            if (store.accumulate)
                v = make_uint4(as_bits(__builtin_fmaf(gate, as_float(v.x), x.x)), as_bits(__builtin_fmaf(gate, as_float(v.y), x.y)),
                               as_bits(__builtin_fmaf(gate, as_float(v.z), x.z)), as_bits(__builtin_fmaf(gate, as_float(v.w), x.w)));
            else if (store.gate)
                v = make_uint4(as_bits(gate * as_float(v.x)), as_bits(gate * as_float(v.y)), as_bits(gate * as_float(v.z)),
                               as_bits(gate * as_float(v.w)));
        }
        uint8_t *at = dst + t * pitch;
        if (ES == 4 && whole_chunks) {
            store_streaming(at, v);
        } else if (ES < 4) {
            *reinterpret_cast<uint4 *>(at) = v;
        } else {                      // 32-bit rows that are not a multiple of 16 bytes
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < live) reinterpret_cast<uint32_t *>(at)[e] = w[e];
        }
    }
};

// Behind a tile's stage buffers: what its outputs need that takes a load each, fetched beside the K loop by direct loads (the
// compiler would wait for a load into registers, and with it for the stages).
//   table : the byte table      dest : output row of every tile row (kScatter with a row list)      gate : its factor
template <class Store, int BM>
struct OutSide {
    static constexpr int ROWS = BM < 64 ? 64 : BM;
    static constexpr int TABLE = 0, DEST = Store::kTableBytes, GATE = DEST + ROWS * 4;
    static constexpr int BYTES = Store::kTableBytes + (Store::kScatter ? ROWS * 8 : 0);
    const Store &store;
    const int32_t *rows;
    long m0, n_rows;
    uint8_t *lds;              // BYTES of its own

    __device__ __forceinline__ long row(int ml) const { return min(m0 + ml, n_rows - 1); }
    __device__ __forceinline__ uint32_t at(int off) const { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds + off; }
    // before the loads of the first stage
    __device__ __forceinline__ void fetch_rows(int wave, int lane) const {
        if constexpr (Store::kTableBytes != 0) {
            if (wave == 0) direct_load_4(static_cast<const uint8_t *>(store.table) + lane * 4, at(TABLE));
        }
        if constexpr (Store::kScatter) {
            if (rows && wave < ROWS / 64) direct_load_4(rows + row(wave * 64 + lane), at(DEST + wave * 256));
        }
    }
    // once those have landed; the wavefront reads what it fetched itself
    __device__ __forceinline__ void fetch_gates(int wave, int lane) const {
        if constexpr (Store::kScatter) {
            if (store.gate && wave < ROWS / 64) direct_load_4(store.gate + dest(wave * 64 + lane), at(GATE + wave * 256));
        }
    }
    // behind a barrier
    __device__ __forceinline__ long dest(int ml) const {
        if constexpr (Store::kScatter)
            if (rows) return (long)reinterpret_cast<const int32_t *>(lds + DEST)[ml];
        return row(ml);
    }
    __device__ __forceinline__ float gate(int ml) const {
        if constexpr (Store::kScatter)
            if (store.gate) return reinterpret_cast<const float *>(lds + GATE)[ml];
        return 1.0f;
    }
};

template <class T, int BM, int BN, int SB, int NS, class Store>
struct NtShape {
    static constexpr int STAGE = (BM + T::kPlanes * BN) * SB;
    // epilogue staging: 32 rows of a wavefront's columns each, 16 bytes apart modulo the banks
    static constexpr int PITCH = BN / 2 * Store::kBytes + 16, SLAB_BYTES = 32 * PITCH;
    static constexpr int OUT_BYTES = 4 * SLAB_BYTES > Store::kHashBytes ? 4 * SLAB_BYTES : Store::kHashBytes;
    static constexpr int RING_BYTES = NS * STAGE > OUT_BYTES ? NS * STAGE : OUT_BYTES;
    // a ring that fills half of a CU's LDS to the last byte: the side loads wait for the ring to be free
    static constexpr bool SIDE_LATE = RING_BYTES == 80 * 1024 && OutSide<Store, BM>::BYTES > 0;
    static constexpr int SIDE_AT = SIDE_LATE ? 4 * SLAB_BYTES : RING_BYTES;
    static constexpr int LDS_BYTES = SIDE_LATE ? RING_BYTES : RING_BYTES + OutSide<Store, BM>::BYTES;
    static_assert(SIDE_AT + OutSide<Store, BM>::BYTES <= LDS_BYTES, "room for the side loads");
};

template <class T, int BM, int BN, int SB, int NS, int LS, bool BLOCKED, class Store>
__device__ __forceinline__ void nt_gemm_tile(const GemmArgs &g, const Store &store, int block, uint8_t *lds, long first_row, long end_row) {
    using S = NtShape<T, BM, BN, SB, NS, Store>;
    constexpr int kStageBytes = SB;                     // bytes of K per stage and row
    constexpr int kChunksPerRow = SB / 16;              // 16-byte chunks per LDS row
    constexpr int KK = SB / 32;                         // 32-byte MFMA steps per stage
    static_assert(SB == 64 || SB == 128, "stage rows of 64 or 128 bytes");
    constexpr int NP = T::kPlanes;
    constexpr int MI = BM / 64, NJ = BN / 64;           // 32x32 tiles per wavefront
    constexpr int A_BYTES = BM * kStageBytes, B_BYTES = BN * kStageBytes;
    constexpr int STAGE = S::STAGE;
    constexpr int ROWS_PER_INSTR = 1024 / kStageBytes;  // LDS rows one wavefront load fills
    constexpr int A_INSTR = BM / ROWS_PER_INSTR / 4;    // loads per wavefront and stage
    constexpr int B_INSTR = BN / ROWS_PER_INSTR / 4;
    constexpr int ES = Store::kBytes;
    constexpr bool PACKED = T::kPacked;
    constexpr int LOADS = A_INSTR + (PACKED ? 0 : NP * B_INSTR);       // direct loads per wavefront and stage
    // Narrow outputs and sign codes: the MFMAs compute the transposed tile (B rows down, A rows across), so that a lane
    // ends up with four consecutive columns of a row: a quarter of the LDS writes on the way out.  With int8 operands
    // the chip then holds about 4 % less of its rate under full load, so 32-bit outputs are computed upright.
    constexpr bool ROWS_ACROSS = ES < 4 || Store::kSignCodes;
    static_assert(NS >= 2 && NS <= 4, "ring of two to four stages");

    const int32_t *rows;
    long n_rows;
    resolve_rows(g.sel, rows, n_rows);
    n_rows = n_rows < end_row ? n_rows : end_row;
    // An XCD's share of the B planes (chosen by the host to fit the L2) stays resident, and each row tile of A is fetched by
    // col_groups L2s only.
    int row_tile, col_tile;
    g.tile_of(block, row_tile, col_tile);
    const long m0 = first_row + (long)row_tile * BM;
    if (m0 >= n_rows || col_tile >= g.col_tiles) return;
    const int n0 = col_tile * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
    const int N = g.N;
    const size_t row_bytes = (size_t)g.K * T::kElemBytes;
    const size_t a_row_bytes = BLOCKED ? 64 : (size_t)(g.a_ld > 0 ? g.a_ld : g.K) * T::kElemBytes;
    const int a_valid_bytes = (g.a_valid > 0 ? g.a_valid : g.K) * T::kElemBytes;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;

    // ---- what each lane fetches.  Wavefront w issues load i for LDS rows
    //      (w * X_INSTR + i) * ROWS_PER_INSTR + lane / kChunksPerRow, physical chunk lane % kChunksPerRow.
    //      Rows past the end are clamped to the last valid row (computed, never stored).
    const uint8_t *a_src[A_INSTR];
#pragma unroll
    for (int i = 0; i < A_INSTR; ++i) {
        const int r = (wave * A_INSTR + i) * ROWS_PER_INSTR + lane / kChunksPerRow;
        const int c = swizzle<kChunksPerRow>(r, lane % kChunksPerRow);
        long m = m0 + r;
        m = m < n_rows ? m : n_rows - 1;
        const long src = (g.gather_a && rows) ? (long)rows[m] : m;
        a_src[i] = static_cast<const uint8_t *>(g.a) + (size_t)src * a_row_bytes + c * 16;
    }
    // The furthest stage offset at which this lane's chunk still lies inside an A row (64-byte stages: every load of
    // a lane has the same physical chunk, rows 16 apart swizzle alike).  Beyond it the lane re-reads the row's last
    // 16 bytes; with whole rows (a_valid == K) no stage offset gets that far.
    int a_klim = 0;
    if constexpr (SB == 64)
        a_klim = a_valid_bytes - 16 - swizzle<kChunksPerRow>(lane / kChunksPerRow, lane % kChunksPerRow) * 16;
    const uint8_t *b_src[NP][B_INSTR];
#pragma unroll
    for (int i = 0; i < B_INSTR; ++i) {
        const int r = (wave * B_INSTR + i) * ROWS_PER_INSTR + lane / kChunksPerRow;
        const int c = swizzle<kChunksPerRow>(r, lane % kChunksPerRow);
        const int n = min(n0 + r, N - 1);
#pragma unroll
        for (int p = 0; p < (PACKED ? 0 : NP); ++p)
            b_src[p][i] = static_cast<const uint8_t *>(g.b[p]) + (size_t)n * row_bytes + c * 16;
    }

    // Packed weights: a thread takes PB bytes of a stage's row, 16 weights per 8 of them: a chunk of either plane.  The bytes of
    // two stages are loaded at once (a row's 64 bytes: half a line, and its other half next time), one stage before the first
    // of them is due.
    constexpr int PB = BN / 8, PPR = 32 / PB;           // bytes of a thread and stage, threads of a row
    static_assert(!PACKED || (SB == 64 && NS == 2 && (PB == 8 || PB == 16)), "packed stages");
    typedef typename std::conditional<PB == 16, uint4, uint2>::type packed_t;
    packed_t packed0, packed1;                          // of an even and the odd stage behind it
    const int p_row = tid / PPR, p_chunk = tid % PPR * (PB / 8);
    const uint8_t *p_src = static_cast<const uint8_t *>(g.b[0]) + (size_t)min(n0 + p_row, N - 1) * (row_bytes / 2) + tid % PPR * PB;
    auto load_packed = [&](int s) {                     // of stages s (even) and s + 1
        packed0 = *reinterpret_cast<const packed_t *>(p_src + s * 32);
        packed1 = *reinterpret_cast<const packed_t *>(p_src + min(s + 1, (int)(row_bytes / 64) - 1) * 32);
    };
    // chunk c of a thread's PB / 8, into both planes of a stage
    auto unpack = [&](packed_t w, int c, int slot) {
        uint32_t x0 = w.x, x1 = w.y, a[4], b[4];
        if constexpr (PB == 16) {
            x0 = c == 0 ? w.x : w.z;
            x1 = c == 0 ? w.y : w.w;
        }
        decode8(x0, a, b);
        decode8(x1, a + 2, b + 2);
        uint8_t *at = lds + slot * STAGE + A_BYTES + p_row * kStageBytes + swizzle<kChunksPerRow>(p_row, p_chunk + c) * 16;
        *reinterpret_cast<uint4 *>(at) = make_uint4(a[0], a[1], a[2], a[3]);
        *reinterpret_cast<uint4 *>(at + B_BYTES) = make_uint4(b[0], b[1], b[2], b[3]);
    };

    const OutSide<Store, BM> side{store, rows, m0, n_rows, lds + S::SIDE_AT};

    // Direct load number q (0 .. LOADS-1) of a stage: A rows first, then the B planes.
    auto issue_load = [&](int q, int buf, int kbyte) {
        const uint32_t base = lds_base + buf * STAGE;
        if (q < A_INSTR) {
            direct_load_16(a_src[q] + (BLOCKED ? (size_t)(kbyte / 64) * g.a_block : SB == 64 ? min(kbyte, a_klim) : kbyte), base + (wave * A_INSTR + q) * 1024);
        } else {
            const int p = (q - A_INSTR) / B_INSTR, i = (q - A_INSTR) % B_INSTR;
            direct_load_16(b_src[p][i] + kbyte, base + A_BYTES + p * B_BYTES + (wave * B_INSTR + i) * 1024);
        }
    };
    auto issue_stage = [&](int buf, int kbyte) {
#pragma unroll
        for (int q = 0; q < LOADS; ++q) issue_load(q, buf, kbyte);
    };

    typename T::Acc acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // fragment read offsets (bytes inside a tile) for the 32-byte steps of a stage.  The swizzle of a row depends
    // on the row number modulo 16 only, so tile i of a wavefront reads at the offset of its tile 0 plus 32 rows * i.
    const int fr = lane & 31, fg = lane >> 5;
    int a_rd[KK], b_rd[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        a_rd[kk] = (wm + fr) * kStageBytes + swizzle<kChunksPerRow>(wm + fr, 2 * kk + fg) * 16;
        b_rd[kk] = (wn + fr) * kStageBytes + swizzle<kChunksPerRow>(wn + fr, 2 * kk + fg) * 16;
    }

    auto read_frags = [&](const uint8_t *A, int kk, uint4 (&af)[MI], uint4 (&bf)[NP][NJ]) {
        const uint8_t *B = A + A_BYTES;
#pragma unroll
        for (int i = 0; i < MI; ++i) af[i] = *reinterpret_cast<const uint4 *>(A + a_rd[kk] + i * 32 * kStageBytes);
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                bf[p][j] = *reinterpret_cast<const uint4 *>(B + p * B_BYTES + b_rd[kk] + j * 32 * kStageBytes);
    };
    // One 32-byte step of MFMAs.  When phase >= 0, the direct loads [phase * LPS, (phase+1) * LPS)
    // of the stage at byte kbyte are issued into ring slot `slot`, evenly spaced between the MFMAs:
    // a wavefront that issues its loads back to back stalls on the full vector-memory queue
    // (about 1 KiB per 16 cycles and CU) and leaves its matrix core idle meanwhile.
    const int n_stages = (int)(row_bytes / kStageBytes);
    constexpr int MFMAS = NP * MI * NJ;
    constexpr int LPS = (LOADS + LS - 1) / LS;          // loads per step
    auto multiply = [&](const uint4 (&af)[MI], const uint4 (&bf)[NP][NJ], auto phase_c, auto more_c, bool more, int slot, int kbyte) {
        constexpr int phase = decltype(phase_c)::value;
        constexpr int MORE = decltype(more_c)::value;      // 1: always, 0: never, -1: `more` decides
        static_for<MFMAS>([&](auto m_c) {
            constexpr int m = decltype(m_c)::value;             // MFMAs issued before this one
            constexpr int p = m / (MI * NJ), i = m / NJ % MI, j = m % NJ;
            acc[i][j] = ROWS_ACROSS ? T::mma(bf[p][j], af[i], acc[i][j]) : T::mma(af[i], bf[p][j], acc[i][j]);
            // loads [m * LPS / MFMAS, (m + 1) * LPS / MFMAS) of this step's share follow MFMA m
            if constexpr (phase >= 0) {
                constexpr int q0 = m * LPS / MFMAS, q1 = (m + 1) * LPS / MFMAS;
                if constexpr (q1 > q0) {
                    __builtin_amdgcn_sched_barrier(0);
                    static_for<q1 - q0>([&](auto d_c) {
                        constexpr int q = phase * LPS + q0 + decltype(d_c)::value;
                        if constexpr (q < LOADS && MORE != 0) {
                            if constexpr (MORE == 1)
                                issue_load(q, slot, kbyte);
                            else if (more)
                                issue_load(q, slot, kbyte);
                        }
                    });
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // packed weights: the stage whose first loads these are is unpacked, a chunk behind every other MFMA
            if constexpr (PACKED && phase == 0 && MORE != 0) {
                constexpr int CHUNKS = PB / 8, c0 = m * CHUNKS / MFMAS, c1 = (m + 1) * CHUNKS / MFMAS;
                const bool odd = (kbyte / kStageBytes) & 1;
                if constexpr (c1 > c0)
                    if (MORE == 1 || more) {
                        packed_t w = packed0;
                        if (odd) w = packed1;
                        unpack(w, c0, slot);
                    }
                if constexpr (m == MFMAS - 1)
                    if (odd && kbyte / kStageBytes + 1 < n_stages && (MORE == 1 || more)) load_packed(kbyte / kStageBytes + 1);
            }
        });
    };

    // Software pipeline over a ring of NS stage buffers, all of them loaded ahead.  The LDS
    // fragment reads of one 32-byte step take about half as long as its MFMAs, so they are issued
    // one step ahead and run under the matrix cores.  The barrier that hands over stage s+1 sits
    // before the last step of stage s: by then every fragment of stage s is in registers, so the
    // slot of stage s is free for stage s+NS, whose loads are spread over that last step and the
    // first LS-1 steps of stage s+1; the first fragments of stage s+1 are read under the MFMAs
    // of the last step.
    static_assert(LS >= 1 && LS <= KK, "loads of a stage are spread over at most one stage of steps");
    uint4 af[2][MI], bf[2][NP][NJ];
    if constexpr (!S::SIDE_LATE) side.fetch_rows(wave, lane);
#pragma unroll
    for (int q = 0; q < NS; ++q)
        if (q < n_stages) issue_stage(q, q * kStageBytes);
    if constexpr (PACKED) {
        load_packed(0);
#pragma unroll
        for (int c = 0; c < PB / 8; ++c) {
            unpack(packed0, c, 0);
            if (n_stages > 1) unpack(packed1, c, 1);
        }
        if (n_stages > 2) load_packed(2);
    }
    // Wait until all but the `later` most recently issued stages of this wavefront's loads have landed.
    auto wait_all_but = [&](int later) {
        if (NS >= 4 && later >= 3)
            wait_loads_in_flight<(NS >= 4 ? 3 : 0) * LOADS>();
        else if (NS >= 3 && later == 2)
            wait_loads_in_flight<(NS >= 3 ? 2 : 0) * LOADS>();
        else if (later == 1)
            wait_loads_in_flight<LOADS>();
        else
            wait_loads_in_flight<0>();
    };
    // this wavefront's loads of stage 0 have landed (later stages may still be in flight)
    wait_all_but((n_stages < NS ? n_stages : NS) - 1);
    if constexpr (!S::SIDE_LATE) side.fetch_gates(wave, lane);
    __syncthreads();                             // ... and everyone's
    read_frags(lds, 0, af[0], bf[0]);
    int buf = 0, prev = NS - 1;                  // ring slots of stage s and of stage s-1
    // One stage.  What depends on the position in the K loop is passed as a compile-time constant where the caller
    // knows it (1 = yes, 0 = no, -1 = decide at run time), so that the steady state has no branch around a load and
    // no branch join in front of the MFMAs (at a join the compiler must assume the longer of the two wait lists):
    //   next : there is a stage s+1 (hand-over barrier and its first fragment reads)
    //   m0   : stage s+NS exists (its first share of loads goes into the slot this stage leaves)
    //   m1   : stage s-1+NS exists and s >= 1 (its further shares go into the slot of stage s-1)
    auto stage = [&](int s, auto next_c, auto m0_c, auto m1_c) {
        constexpr int NEXT = decltype(next_c)::value, M0 = decltype(m0_c)::value, M1 = decltype(m1_c)::value;
        const bool next = NEXT < 0 ? s + 1 < n_stages : NEXT != 0;
        const bool m0 = M0 < 0 ? s + NS < n_stages : M0 != 0;
        const bool m1 = M1 < 0 ? (s >= 1 && s - 1 + NS < n_stages) : M1 != 0;
        const uint8_t *cur = lds + buf * STAGE;
        const int nxt = buf + 1 == NS ? 0 : buf + 1;
        static_for<KK>([&](auto kk_c) {
            constexpr int kk = decltype(kk_c)::value;
            if constexpr (kk + 1 < KK) {
                read_frags(cur, kk + 1, af[(kk + 1) & 1], bf[(kk + 1) & 1]);
            } else if (next) {
                // stage s+1 has landed (this wavefront's part); stages s+2 .. s+NS-1 may still be in flight
                if constexpr (M0 == 1)
                    wait_all_but(NS - 2);
                else
                    wait_all_but((s + NS - 1 < n_stages ? s + NS - 1 : n_stages - 1) - (s + 1));
                __syncthreads();                 // everyone's has, and everyone holds its last fragments of stage s
                read_frags(lds + nxt * STAGE, 0, af[0], bf[0]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kk == KK - 1) {
                // first share of stage s+NS, into the slot this stage has just left
                multiply(af[kk & 1], bf[kk & 1], std::integral_constant<int, 0>{}, m0_c, m0, buf, (s + NS) * kStageBytes);
            } else if constexpr (kk + 1 < LS) {
                // further shares of stage s-1+NS, into the slot of stage s-1
                multiply(af[kk & 1], bf[kk & 1], std::integral_constant<int, kk + 1>{}, m1_c, m1, prev, (s - 1 + NS) * kStageBytes);
            } else {
                multiply(af[kk & 1], bf[kk & 1], std::integral_constant<int, -1>{}, std::integral_constant<int, 0>{}, false, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        prev = buf;
        buf = nxt;
    };
    using Yes = std::integral_constant<int, 1>;
    using No = std::integral_constant<int, 0>;
    using Ask = std::integral_constant<int, -1>;
    if (n_stages > NS + 1) {
        int s = 0;
        stage(s++, Yes{}, Yes{}, No{});
        for (; s < n_stages - NS; ++s) stage(s, Yes{}, Yes{}, Yes{});
        stage(s++, Yes{}, No{}, Yes{});
        for (; s < n_stages - 1; ++s) stage(s, Yes{}, No{}, No{});
        stage(s, No{}, No{}, No{});
    } else {
        for (int s = 0; s < n_stages; ++s) stage(s, Ask{}, Ask{}, Ask{});
    }

    // Transposed tile: accumulator register r of lane l holds row l % 32, column 8 (r / 4) + 4 (l / 32) + r % 4.
    // ---- sign codes: a wavefront's columns are one code word of a head or half of one; each half-wavefront has every
    //      other nibble.
    if constexpr (Store::kSignCodes) {
        if (n0 < store.code_cols) {               // uniform per workgroup
            static_assert(NJ <= 2, "a wavefront's columns lie inside one code word");
            const int col0 = n0 + wn;
            if constexpr (Store::kHashBytes != 0) {
                static_assert(NJ == 2, "a wavefront has all columns of a head");
                return store.hash(acc, lds, m0 + wm, n_rows, col0, tid);
            }
            const int part = col0 / store.part_width;
            const int cin = col0 - part * store.part_width;
            const int head = cin / store.head_dim, w = (cin % store.head_dim) / 64, W = store.head_dim / 64;
            uint64_t *dst = part == 0 ? store.codes[0] : store.codes[1];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                uint32_t word[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    uint32_t neg = 0;
#pragma unroll
                    for (int r = 15; r >= 0; --r) {
                        neg = __builtin_amdgcn_alignbit(neg, (uint32_t)acc[i][j][r], 31);      // neg << 1 | sign
                        if (r % 4 == 0 && r > 0) neg <<= 4;
                    }
                    neg <<= 4 * fg;
                    word[j] = ~(neg | (uint32_t)__shfl_xor((int)neg, 32));
                }
                const long m = m0 + wm + i * 32 + fr;
                if (fg == 0 && m < n_rows) {
                    const long b = m / store.tokens, n = m % store.tokens;
                    uint64_t *at = dst + ((size_t)(b * store.heads + head) * store.tokens + n) * W + w;
                    if constexpr (NJ == 2)
                        *at = word[0] | ((uint64_t)word[NJ - 1] << 32);
                    else
                        reinterpret_cast<uint32_t *>(at)[cin / 32 & 1] = word[0];
                }
            }
            return;
        }
    }

    // ---- epilogue.  Every wavefront turns 32 rows of its columns at a time into rows of 16-byte chunks, through LDS of
    //      its own.  Staging 64 rows of the workgroup's whole tile took two barriers per 32 rows of a wavefront and one
    //      LDS write per element: 98304 x 1024 <- 256 int8 to int8 75 -> 64 us, 12608 x 1536 <- 384 28 -> 25 us.
    constexpr int PITCH = S::PITCH, CPR = BN / 2 * ES / 16;       // 16-byte chunks of a staged row
    constexpr int NC = CPR / 2, ROWS_PER_CHUNK = 64 / CPR;        // chunks of a lane per 32 rows, and the rows between them
    uint8_t *slab = lds + wave * S::SLAB_BYTES;
    const uint8_t *table = side.lds;
    const int cc = lane % CPR, cr = lane / CPR;                   // this lane's chunk of a row, its first row
    const ChunkOut<Store> chunk(store, n0 + wn + cc * (16 / ES), N);
    // late: the row's addresses are made where they are used.  Made ahead for all rows, beside a residual on its way, they took more registers than
    // there are (30000 x 768 <- 768 with a residual, 128 x 128 tiles, 44 spilled: 84.5 us, 54.3 so; 60000 x 384 <- 384 70.7, 40.4).
    auto row_of = [&](int i, int q, bool late) {
        int r = cr;
        if (late) asm volatile("" : "+v"(r));
        return wm + i * 32 + q * ROWS_PER_CHUNK + r;
    };
    wait_loads_in_flight<0>();
    __syncthreads();                              // the last stage has been read, `side` is complete
    if constexpr (S::SIDE_LATE) {
        side.fetch_rows(wave, lane);
        wait_loads_in_flight<0>();
        side.fetch_gates(wave, lane);
        wait_loads_in_flight<0>();
        __syncthreads();
    }
    // Table lookups run one 32x32 tile ahead of the packing: four at a time, each four waited out the LDS's latency (131072 x
    // 1024 <- 256: 4.5 us per 256 x 128 tile, longer than its products).
    constexpr int AHEAD = Store::kTableBytes != 0 ? 1 : 0;
    uint32_t conv[1 + AHEAD][16];
    auto convert = [&](auto t_c) {
        constexpr int t = decltype(t_c)::value, i = t / NJ, j = t % NJ;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int nl = j * 32 + (ROWS_ACROSS ? 8 * (r / 4) + 4 * fg + r % 4 : fr);
            conv[t & AHEAD][r] = store.convert(acc[i][j][r], min(n0 + wn + nl, N - 1), table);
        }
    };
    // With nothing to read for the outputs, no registers are kept for it: 131072 x 256 <- 1024 was 87 us with them, 82 without.
    auto emit = [&](auto reads_c) {
        constexpr bool READS = decltype(reads_c)::value;
        float4 ext[READS ? 2 : 1][NC];
        auto fetch = [&](int i) {
#pragma unroll
            for (int q = 0; q < NC; ++q) ext[READS ? i & 1 : 0][q] = READS ? chunk.fetch(side.dest(row_of(i, q, Store::kLinear && READS))) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        };
        fetch(0);
        if constexpr (AHEAD) convert(std::integral_constant<int, 0>{});
        static_for<MI * NJ>([&](auto t_c) {
            constexpr int t = decltype(t_c)::value, i = t / NJ, j = t % NJ;
            if constexpr (t + AHEAD < MI * NJ) convert(std::integral_constant<int, t + AHEAD>{});
            if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);
            const uint32_t(&v)[16] = conv[t & AHEAD];
            if constexpr (ROWS_ACROSS) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint8_t *at = slab + fr * PITCH + (j * 32 + 8 * q + 4 * fg) * ES;
                    if constexpr (ES == 1)
                        *reinterpret_cast<uint32_t *>(at) = (v[4 * q] | (v[4 * q + 1] << 8)) | ((v[4 * q + 2] | (v[4 * q + 3] << 8)) << 16);
                    else if constexpr (ES == 2)
                        *reinterpret_cast<uint2 *>(at) = make_uint2(v[4 * q] | (v[4 * q + 1] << 16), v[4 * q + 2] | (v[4 * q + 3] << 16));
                    else
                        *reinterpret_cast<uint4 *>(at) = make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
                }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    *reinterpret_cast<uint32_t *>(slab + mfma32_row(r, lane) * PITCH + (j * 32 + fr) * 4) = v[r];
            }
            if constexpr (j == NJ - 1) {                  // 32 rows are complete
                if constexpr (i + 1 < MI) fetch(i + 1);
#pragma unroll
                for (int q = 0; q < NC; ++q) {
                    const int ml = row_of(i, q, Store::kLinear && READS);
                    const uint4 c = *reinterpret_cast<const uint4 *>(slab + (q * ROWS_PER_CHUNK + cr) * PITCH + cc * 16);
                    if (m0 + ml < n_rows && chunk.live > 0) chunk.put(c, ext[READS ? i & 1 : 0][q], side.gate(ml), side.dest(ml));
                }
            }
        });
    };
    if constexpr (ChunkOut<Store>::MAY_READ) {
        if (chunk.reads()) return emit(std::true_type{});
    }
    emit(std::false_type{});
}

// A tile shape as launch_tile and the kernels below take it.
template <class T, int BM_, int BN_, int SB, int NS, int LS, bool BLOCKED = false>
struct NtTile {
    static_assert(!BLOCKED || SB == 64, "columns of a stage");
    static constexpr int BM = BM_, BN = BN_;
    template <class Store>
    static constexpr int lds_bytes() { return NtShape<T, BM, BN, SB, NS, Store>::LDS_BYTES; }
    template <class Store>
    __device__ static __forceinline__ void run(const GemmArgs &g, const Store &store, int block, uint8_t *lds, long first_row = 0,
                                               long end_row = 0x7fffffffL) {       // of the selected rows, those that a launch gives to these tiles
        nt_gemm_tile<T, BM, BN, SB, NS, LS, BLOCKED, Store>(g, store, block, lds, first_row, end_row);
    }
    // The fewest column groups whose share of the B planes stays resident in a 4 MiB L2 next to
    // the A rows streaming through it.  (Fewer groups fetch fewer bytes when A is the larger operand,
    // but a B share that is evicted between row tiles costs more time than the extra A traffic.)  More groups where the L2s
    // fetch less in all with them, A col_groups times and B 8 / col_groups times: with few rows that fetch is what takes the time
    // (3152 x 3072 <- 768 27.6 -> 25.3 us, 2600 x 1536 <- 384 10.0 -> 8.8, 4000 x 1024 <- 1024 14.8 -> 13.7; block of 2364 tokens x
    // 768 70.4 -> 65.4, layer of 1379 84.1 -> 83.3).  Not where rows of 32-bit outputs are no whole 128-byte lines: tiles beside each
    // other then write the same lines from different L2s, and the last columns are shared out less evenly (5932 x 1784 <- 32 12.9 ->
    // 17.3, 8393 x 1316 <- 192 18.6 -> 21.5; of 212 such shapes 60 lost more than 3 % and 37 gained it, of 61 others 1 and 12).
    static int col_groups(const GemmArgs &g) {
        const size_t b_bytes = T::kPacked ? (size_t)g.N * g.K / 2 : (size_t)T::kPlanes * g.N * g.K * T::kElemBytes;
        int cg = 1;
        while (cg < 8 && b_bytes / cg > (size_t)(5 << 19)) cg *= 2;     // 2.5 MiB
        const long col_tiles = (g.N + BN - 1) / BN;
        const double a_bytes = (double)g.sel.max_rows * g.K * T::kElemBytes;
        while (g.N % 32 == 0 && cg < 8 && 2 * cg <= col_tiles && a_bytes * cg < b_bytes * (4.0 / cg)) cg *= 2;
        return cg;
    }
};

// Workgroups that cover n_rows x N with this tile (a multiple of 8: one share per XCD).
template <class Tile>
__host__ __device__ inline long tile_blocks(long n_rows, const GemmArgs &g) {
    const long row_tiles = (n_rows + Tile::BM - 1) / Tile::BM;
    const int log_rg = 3 - g.log_groups;
    return 8 * ((row_tiles + (1 << log_rg) - 1) >> log_rg) * g.cols_per_group;
}

template <class Tile, int OCC, class Store>
__global__ __launch_bounds__(256, OCC) void gemm_kernel(GemmArgs g, Store store) {
    constexpr int LDS_BYTES = Tile::template lds_bytes<Store>();
    static_assert(LDS_BYTES * OCC <= 160 * 1024, "OCC workgroups of this tile do not fit the LDS of a CU");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_BYTES];
    Tile::template run<Store>(g, store, blockIdx.x, lds);
}

template <class Tile, int OCC, class Store>
int launch_tile(const GemmArgs &g, const Store &store, hipStream_t st, const char *what) {
    GemmArgs ga = g;
    ga.share_out(Tile::BN, Tile::col_groups(g));
    const long blocks = tile_blocks<Tile>(g.sel.max_rows, ga);
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "%s: too many tiles for one launch", what);
    gemm_kernel<Tile, OCC, Store><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(ga, store);
    return check_launch(what);
}

// How many rows go to tiles of BM rows where tiles of half of them take the others: those of as many tiles as every CU has at least, if all
// tiles are one round of workgroups (OCC a CU, which share its matrix cores) and no more than every other CU would have one more.  The CUs
// then end half a tile apart instead of a whole one.  rest: tiles of an XCD that other rows have.  All rows: no gain.
template <int BM, int OCC>
__host__ __device__ inline uint32_t even_rows(uint32_t n_rows, const GemmArgs &g, uint32_t rest) {
    constexpr uint32_t CUS = 32;                             // of an XCD
    const uint32_t log_rg = 3 - g.log_groups, cols = g.cols_per_group;
    auto rows_of = [&](uint32_t n, uint32_t bm) { return ((n + bm - 1) / bm + (1u << log_rg) - 1) >> log_rg; };
    const uint32_t all = rows_of(n_rows, BM) * cols + rest, each = all / CUS * CUS;
    if (all > OCC * CUS || all - each - 1 >= CUS / 2 || each <= rest) return n_rows;
    const uint32_t left = g.by_cols(each - rest), high = (left << log_rg) * BM;          // left: rows of tiles that stay
    if (left == 0 || high >= n_rows) return n_rows;
    const uint32_t low = rows_of(n_rows - high, BM / 2) * cols, room = each - rest - left * cols;
    return low <= CUS + 2 * room && rest + left * cols + low <= OCC * CUS ? high : n_rows;
}

// The fewest tiles an XCD has of n rows, some of which s and the others m takes, with BM_S and BM_M rows to a tile.
template <int BM_S, int BM_M>
long least_tiles(const GemmArgs &s, const GemmArgs &m, long n) {
    auto of = [&](const GemmArgs &g, long bm) { const long span = bm << (3 - g.log_groups); return (n * g.cols_per_group + span - 1) / span; };
    return std::min(of(s, BM_S), of(m, BM_M));
}

// Whether even_rows takes rows from s for some share of n rows (m has the others, rest tiles of BM_M rows).  Where it never does,
// workgroups need not ask: two-expert Linears of 12571 to 99963 tokens, K = 64 3.6 %, 192 1.0 %, 256 0.9 %, 384 and 768 0.3 % on
// average, layers of 5000 to 25000 tokens 0.2 to 0.5 %, blocks 0.1 to 0.3 % (single shapes within 2 % either way).
template <int BM_S, int BM_M, int OCC>
bool may_be_even(const GemmArgs &s, const GemmArgs &m, long n) {
    constexpr long CUS = 32;
    if (least_tiles<BM_S, BM_M>(s, m, n) > OCC * CUS) return false;
    const long span_s = (long)BM_S << (3 - s.log_groups), span_m = (long)BM_M << (3 - m.log_groups);      // rows of a row of tiles in every XCD
    for (long i = 1; i * s.cols_per_group <= OCC * CUS && (i - 1) * span_s < n; ++i) {                   // s has i rows of tiles in the fullest XCD
        const long fewest = std::max(0L, n - i * span_s), most = n - (i - 1) * span_s - 1;               // rows left for m
        for (long j = (fewest + span_m - 1) / span_m; j <= (most + span_m - 1) / span_m; ++j) {
            const long rest = j * m.cols_per_group, all = i * s.cols_per_group + rest, over = all % CUS;
            if (all <= OCC * CUS && over > 0 && over <= CUS / 2 && all - over > rest) return true;
        }
    }
    return false;
}

// The last rows in tiles of half the height (even_rows).  us, without and with: packed weights 12608 x 384 <- 1536 22.7, 20.8, 9000 x 512 <- 1024
// 16.6, 15.1, 25088 x 192 <- 1024 16.8, 15.3, 12608 x 384 <- 384 8.7, 8.3; prepared, with a residual, 12608 x 384 <- 768 15.0, 13.7.  Both experts
// 11000 x 768 <- 768 31.7, 28.4, 7000 x 1152 <- 768 31.7, 28.9, 25088 x 384 <- 384 25.5, 23.6, 12608 x 768 <- 768, 70 % 32.2, 31.3; where no rows are
// taken within 1 % (a workgroup works that out).  Not the tiles of long rows, two a CU (12608 x 384 <- 2304 34.2, 34.5), nor the finer pairs of
// tiles (7000 x 512 <- 512 15.6, 16.1).
template <class Tile, class Low, int OCC, class Store>
__global__ __launch_bounds__(256, OCC) void gemm_even_kernel(GemmArgs g, Store store, int high_blocks, int high_rows) {
    constexpr int LDS_H = Tile::template lds_bytes<Store>(), LDS_L = Low::template lds_bytes<Store>(), LDS_BYTES = LDS_H > LDS_L ? LDS_H : LDS_L;
    static_assert(LDS_BYTES * OCC <= 160 * 1024 && Low::BN == Tile::BN && 2 * Low::BM == Tile::BM, "half of a tile, OCC of either to a CU");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_BYTES];
    if ((int)blockIdx.x < high_blocks) return Tile::template run<Store>(g, store, blockIdx.x, lds, 0, high_rows);
    Low::template run<Store>(g, store, (int)blockIdx.x - high_blocks, lds, high_rows);
}

template <class Tile, class Low, int OCC, class Store>
int launch_even(const GemmArgs &g, const Store &store, hipStream_t st, const char *what) {
    GemmArgs ga = g;
    ga.share_out(Tile::BN, Tile::col_groups(g));
    const long n = g.sel.max_rows, high = g.sel.counts || n >= (1L << 30) ? n : (long)even_rows<Tile::BM, OCC>((uint32_t)n, ga, 0);
    if (high >= n) return launch_tile<Tile, OCC>(g, store, st, what);
    const long high_blocks = tile_blocks<Tile>(high, ga), blocks = high_blocks + tile_blocks<Low>(n - high, ga);      // (of one round)
    gemm_even_kernel<Tile, Low, OCC, Store><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(ga, store, (int)high_blocks, (int)high);
    return check_launch(what);
}

}  // namespace sa

#include "gemm_slice.h"

namespace sa {

// Tile choice, from sweeps over (K, N) of the transformer widths 64 .. 3072 and 50 .. 25088 rows on one MI355X.
// t32, t64: tiles of 32 x 64 and 64 x 64 outputs.
//  * t32 <= 256: not every CU gets a 32 x 64 tile, so the time is that of one tile: gemm_slice.h with 32 rows
//    (965 x 192 <- 768 int8: 4.8 us against 9.5 with 128 x 128 tiles; 197 x 768 <- 3072: 8.7 against 21).  Whole-line stages
//    with up to three 32 x 32 tiles for four CUs: those, whose planes are there in half the time (197 x 768 <- 768 int8 4.9 ->
//    4.2 us, 197 x 768 <- 3072 8.9 -> 6.8, 1000 x 192 <- 768 4.9 -> 4.2; 320 x 768 <- 768, fifteen for sixteen: 5.0 both);
//  * t64 <= 640: up to two and a half 64 x 64 tiles per CU (965 x 768 <- 3072 int8: 11.8 us against 35 with the
//    256 x 128 tiles, 3152 x 768 <- 768: 11.7 against 12.2; fp16 with long rows only up to 320: the next tile up
//    catches up there).  Short rows take 64-byte stages: with few stages the finer ones start sooner
//    (1379 x 1024 <- 256 int8: 5.7 us against 6.1);
//  * beyond, the tiles of this file.  int8 rows of 2 KiB and more in whole 128-byte lines: 128 x 64, 128-byte stages, two
//    per CU (with a residual, 8826 x 768 <- 3072: 53 us against 61 with 256 x 128 tiles, of which 210 leave 46 CUs idle);
//    beyond 1536 tiles of 128 x 128 (six rounds of 128 x 64), 192 x 128 with 64-byte stages.  768 <- 3072 with a residual,
//    128 x 64 against 192 x 128: 25600 rows 123 against 135 us, 64000 rows 345 against 303; from 1400 to 2000 tiles it
//    depends on whose last round is fuller (29824 rows 141 against 133, 36224 rows 164 against 175).  Other int8 rows:
//    128 x 64, three per CU with a ring of three, where 128 x 128 tiles would not fill the chip once or half of their
//    columns would be padding (with a residual, 16384 x 256 <- 1024: 18.9 against 23.8; 12608 x 384 <- 384: 15.9
//    against 21.0); else 256 x 128 (two per CU) or 128 x 128 (three per CU) with 64-byte stages;
//    they do the same work per CU and second, so the one whose last round of workgroups is fuller
//    (12608 x 1536 <- 384: 38 against 29 us; 12608 x 3072 <- 768: 76 against 82).  fp16: long rows 128 x 128 with a
//    ring of three; rows of more than 768 bytes 192 x 128, both one per CU; short rows 128 x 128 with 64-byte stages.
// A row count that lives on the device is taken to be half of its bound (two experts share the tokens).
// Narrow (1- and 2-byte) output rows must be whole 16-byte chunks; operand rows must be a
// multiple of 64 bytes long.
template <class T, class Store>
int launch_gemm(const GemmArgs &g, const Store &store, hipStream_t st, const char *what) {
    if (g.sel.max_rows == 0 || g.N == 0) return SA_OK;
    const size_t row_bytes = (size_t)g.K * T::kElemBytes;
    SA_REQUIRE(row_bytes % 64 == 0 && row_bytes > 0, SA_ERR_SHAPE, "%s: rows of %zu bytes are not a multiple of 64", what, row_bytes);
    const bool short_a = g.a_valid > 0 && g.a_valid != g.K;
    SA_REQUIRE(!short_a || (T::kPlanes == 2 && g.a_valid > 0 && g.a_valid < g.K && g.a_valid % 16 == 0), SA_ERR_SHAPE,
               "%s: A rows of %d valid elements in a contraction of %d", what, g.a_valid, g.K);
    SA_REQUIRE(Store::kBytes == 4 || (size_t)g.N * Store::kBytes % 16 == 0, SA_ERR_SHAPE,
               "%s: narrow output rows of %d elements are not whole 16-byte chunks", what, g.N);
    const bool lines = row_bytes % 128 == 0 && !short_a, long_rows = row_bytes >= 2048;
    const bool counted = g.sel.counts != nullptr;
    const long m_est = counted ? (g.sel.max_rows + 1) / 2 : g.sel.max_rows;
    auto tiles = [&](long bm, long bn) { return ((m_est + bm - 1) / bm) * ((g.N + bn - 1) / bn); };
    const bool whole_line_stages = lines && row_bytes >= 512;
    if constexpr (T::kPlanes == 2) {
        if constexpr (!Store::kSignCodes)
            if (whole_line_stages && tiles(32, 32) <= 192) return launch_tile<SliceTile<T, 1, 1, 128, 5>, 1>(g, store, st, what);
        if (tiles(32, 64) <= 256)
            return whole_line_stages ? launch_tile<SliceTile<T, 1, 2, 128, 4>, 1>(g, store, st, what)
                                     : launch_tile<SliceTile<T, 1, 2, 64, 7>, 1>(g, store, st, what);
        if (tiles(64, 64) <= 640)
            return whole_line_stages ? launch_tile<SliceTile<T, 2, 2, 128, 3>, 1>(g, store, st, what)
                                     : launch_tile<SliceTile<T, 2, 2, 64, 6>, 1>(g, store, st, what);
        if (lines && long_rows)
            return tiles(128, 128) <= 1536 ? launch_tile<NtTile<T, 128, 64, 128, 2, 2>, 2>(g, store, st, what)
                                           : launch_tile<NtTile<T, 192, 128, 64, 2, 1>, 2>(g, store, st, what);
        if (tiles(128, 128) <= 768 || g.N <= 64) return launch_even<NtTile<T, 128, 64, 64, 3, 1>, NtTile<T, 64, 64, 64, 3, 1>, 3>(g, store, st, what);
        const long rounds256 = (tiles(256, 128) + 511) / 512, rounds128 = (tiles(128, 128) + 767) / 768;
        const bool wide = counted ? ((g.sel.max_rows + 255) / 256) * ((g.N + 127) / 128) >= 512    // no rounds to speak of
                                  : rounds256 * 5 <= rounds128 * 4;      // a round of the larger tiles takes 1.25 times as long
        if (wide) return launch_tile<NtTile<T, 256, 128, 64, 2, 1>, 2>(g, store, st, what);
        return launch_tile<NtTile<T, 128, 128, 64, 2, 1>, 3>(g, store, st, what);
    } else {
        if (whole_line_stages && tiles(32, 32) <= 192) return launch_tile<SliceTile<T, 1, 1, 128, 8>, 1>(g, store, st, what);
        if (tiles(32, 64) <= 256)
            return whole_line_stages ? launch_tile<SliceTile<T, 1, 2, 128, 6>, 1>(g, store, st, what)
                                     : launch_tile<SliceTile<T, 1, 2, 64, 8>, 1>(g, store, st, what);
        if (tiles(64, 64) <= (long_rows ? 320 : 640))
            return whole_line_stages ? launch_tile<SliceTile<T, 2, 2, 128, 4>, 1>(g, store, st, what)
                                     : launch_tile<SliceTile<T, 2, 2, 64, 9>, 1>(g, store, st, what);
        if (lines && long_rows) return launch_tile<NtTile<T, 128, 128, 128, 3, 2>, 1>(g, store, st, what);
        if (lines && row_bytes > 768) return launch_tile<NtTile<T, 192, 128, 128, 2, 2>, 1>(g, store, st, what);
        return launch_tile<NtTile<T, 128, 128, 64, 3, 1>, 2>(g, store, st, what);
    }
}

// The same on packed weights, without the launch that decodes them (3 to 5 us): whether that is faster for max_rows rows (as
// launch_gemm estimates them), and the launch.  A stage's weights come in as 32 bytes of a row instead of 128, which in the
// K loop pays for their decoding; of the tiles those that leave registers for it (below: decode and planes, packed 128 x 64, packed
// 192 x 128; us):
//  * 192 x 128, two per CU, for rows of 768 bytes and more where that is the fuller way (packed_tall);
//  * 128 x 64, three per CU (12608 x 1536 <- 384 33.5, 27.1, 31.5; 12608 x 384 <- 1536 25.9, 23.1, 23.0; 100000 x 256 <- 64 27, 20.5;
//    3000 x 1024 <- 1024 16, 13.5);
//  * where gemm_slice.h would take the planes, 64 x 64 for rows up to 1024 bytes (1379 x 3072 <- 768 22 -> 15; 965 x 768 <-
//    3072 18 -> 21.6: those stay).
// The planes stay
//  * beyond 2^35 multiply-adds, 2^34 for rows of less than 768 bytes, where the decode is no longer worth its removal (65000 x
//    3072 <- 768 333 against 346, 131072 x 256 <- 1024 86 against 89, 50000 x 1536 <- 384 87.9 against 92.8);
//  * for rows of 2 KiB and more that do not fill 192 x 128 tiles (11000 x 768 <- 3072 64.7 against 72.6; 25088 x 512 <- 2048 61.6
//    against 68.4), or of which only the device knows how many there are, so that the tiles are chosen for half of them (768 <-
//    3072, 8826 of 12608 rows 51.4 against 55.1, 17561 of 25088 91 against 100; 3072 <- 768 of the same 53.4 against 48.8 and 91.5
//    against 86.3, 384 <- 1536 23.4 against 23.7);
//  * for rows of 1 KiB and more that do not, but make more than a round of the larger tiles of the planes (40000 x 384 <- 1536 47.2,
//    58.1, 55.8; 50000 x 384 <- 1536 69.4, 74.0, 72.5; 131072 x 256 <- 1024 73.9, 83.8, 80.3; 32000 x 1024 <- 1024 74.7, 81.4, 77.6);
//    where half of the last tile's columns would be padding, only with no more than one (40000 x 320 <- 1280 40.6, 43.0, 46.7;
//    50000 x 320 <- 1280 55.2, 50.2, 59.7);
//  * for rows up to 256 bytes with many outputs in rows that are no whole 128-byte lines, of which narrower tiles share more (planes,
//    packed: 232794 x 116 <- 64 41.7, 52.5; 18272 x 1836 <- 128 50.8, 60.1; 48347 x 748 <- 256 56.2, 61.6; 53086 x 589 <- 64 52.8, 55.2;
//    5831 x 3220 <- 192 34.3, 38.4; with fewer 8 to 13 % for packed on average);
//  * for less than 64 columns and rows of 768 bytes and more, where the tile is mostly padding (93878 x 37 <- 768 21.3, 25.5; 185423 x
//    10 <- 896 31.4, 33.9; 77000 x 64 <- 768 19.0, 16.0).
// 192 x 128 tiles: an XCD takes 32 of them, one on each CU, and 32 more beside those in not much more time.  The fullest XCD's come
// in `halves` of 32, and all eight XCDs lack `lack` tiles to fill as many:
//  * the second half to run beside a first may lack 20 (12608 x 768 <- 768, 50 of 64: 26.3, 23.1, 22.6; 25088 x 384 <- 1536, 49: 42.1,
//    40.2, 36.3; 16000 x 512 <- 1024, 42: 24.7, 21.7, 25.9);
//  * the third, alone behind two others, 10 (45000 x 384 <- 1536, 88 of 96: 62.7, 66.6, 57.1; 65536 x 256 <- 1024, 86: 39.7, 42.2, 41.6);
//  * the fourth 22 (28000 x 768 <- 768, 110 of 128: 46.7, 43.3, 41.9; 25088 rows, 98: 39.2, 39.1, 41.2);
//  * the fifth and sixth 30 with rows of less than 1 KiB (80000 x 384 <- 768, 156 of 160: 60.8, 63.2, 56.9; 65536 rows, 128: 51.2, 48.9,
//    52.8; 14500 x 2304 <- 768, 171 of 192: 71.6, 67.9, 63.3; 40000 x 768 <- 768, 157: 59.3, 60.5, 62.3), else any and 17 (25088 x 1024
//    <- 1024, 131 of 160: 70.0, 66.8, 67.6; 65536 x 512 <- 1024, 171 of 192: 74.2, 84.3, 80.8);
//  * from the seventh on any (25088 x 1536 <- 768: 78.7, 76.0, 73.9).
// Where half of the last tile's columns would be padding only up to four halves, and less (32000 x 320 <- 1280, 63 of 64: 35.9, 34.9,
// 32.6; 25088 rows, 49: 29.7, 25.9, 30.6; 60000 rows, 117 of 128: 63, 62.0, 59.8; 80000 x 192 <- 768, 104 of 128: 37.5, 33.3, 43.0).
inline bool packed_tall(long m_est, int N, int K) {
    const long row_tiles = (m_est + 191) / 192, col_tiles = (N + 127) / 128;
    const long halves = ((row_tiles + 7) / 8 * col_tiles + 31) / 32, lack = 256 * halves - row_tiles * col_tiles;      // of all XCDs
    if (K < 768 || N <= 64 || halves < 2) return false;
    if (N % 128 > 0 && N % 128 <= 64) return halves == 3 ? N > 256 && lack <= 8 * 6 : lack <= 8 * 12 && halves <= (N > 256 ? 4 : 2);
    switch (halves) {
        case 2: return lack <= 8 * 20;
        case 3: return lack <= 8 * 10;
        case 4: return lack <= 180;
        case 5: return K >= 1024 || lack <= 8 * 30;
        case 6: return lack <= 8 * (K >= 1024 ? 17 : 30);
    }
    return true;
}

inline bool packed_gemm(long max_rows, bool counted, int N, int K) {
    const long m_est = counted ? (max_rows + 1) / 2 : max_rows;
    auto tiles = [&](long bm, long bn) { return ((m_est + bm - 1) / bm) * ((N + bn - 1) / bn); };
    if (K % 64 != 0 || (double)m_est * N * K > (K < 768 ? 17179869184.0 : 34359738368.0)) return false;
    if (tiles(64, 64) <= 640) return K <= 1024;
    if ((N < 64 && K >= 768) || (N % 32 != 0 && K <= 256 && m_est * N >= 15 << 20)) return false;
    if (packed_tall(m_est, N, K)) return K < 2048 || !counted;
    if (K >= 2048) return false;
    const bool padded = N % 128 > 0 && N % 128 <= 64;
    return !(K >= 1024 && tiles(128, 128) > 768 && (!padded || tiles(256, 128) <= 512));
}

template <class Store>
int launch_gemm_packed(const GemmArgs &g, const Store &store, hipStream_t st, const char *what) {
    typedef I8PackedTraits T;
    if (g.sel.max_rows == 0 || g.N == 0) return SA_OK;
    SA_REQUIRE(g.K % 64 == 0 && g.K > 0 && (Store::kBytes == 4 || (size_t)g.N * Store::kBytes % 16 == 0), SA_ERR_SHAPE,
               "%s: rows of %d and outputs of %d", what, g.K, g.N);
    const long m_est = g.sel.counts ? (g.sel.max_rows + 1) / 2 : g.sel.max_rows;
    auto tiles = [&](long bm, long bn) { return ((m_est + bm - 1) / bm) * ((g.N + bn - 1) / bn); };
    if (tiles(64, 64) <= 640) return launch_tile<NtTile<T, 64, 64, 64, 2, 1>, 4>(g, store, st, what);
    if (packed_tall(m_est, g.N, g.K)) return launch_tile<NtTile<T, 192, 128, 64, 2, 1>, 2>(g, store, st, what);
    return launch_even<NtTile<T, 128, 64, 64, 2, 1>, NtTile<T, 64, 64, 64, 2, 1>, 3>(g, store, st, what);
}

}  // namespace sa
