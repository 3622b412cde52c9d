// The matrix-core GEMM of gemm_mfma.h for problems whose 128- and 256-row tiles would leave most of the chip idle:
//     C[m, n] = sum_p sum_k A[m, k] * B_p[n, k]
//
// What bounds such a problem is not the matrix cores but how long one tile takes to come in: a CU fills its LDS
// from the L2 at about 54 bytes per clock, and a K loop with two stage buffers waits out the L2's latency at every
// stage.  So the tile is small (enough tiles that every CU has one), the four wavefronts of a workgroup share it by
// splitting every stage of K between them (wavefront w multiplies 32-byte step w of the stage; each holds the whole
// tile's accumulators, so a stage needs no more LDS reads than one wavefront's fragments), and the ring of stage
// buffers is deep: NS - 1 stages of whole 128-byte lines are in flight at once, with one barrier per stage.
// The four partial tiles meet in LDS in ascending order (integers: any order; floats: always the same one).
// Measured (MI355X, 965 rows x 768 <- 3072, two int8 planes, alone): 11.8 us against 35 us with 256 x 128 tiles;
// 197 rows x 768 <- 3072: 6.8 us with 32 x 32 tiles and 8.9 with 32 x 64 against 21 us with 128 x 128 tiles.
#pragma once

namespace sa {

// Accumulators of one 32-bit element as the tiles keep them in LDS.
template <class T>
struct AccElem;
template <>
struct AccElem<I8Traits> { typedef int32_t type; };
template <>
struct AccElem<F16Traits> { typedef float type; };

template <class T, int MI, int NJ, int SB, int NS, class Store>
struct SliceShape {
    static constexpr int BM = 32 * MI, BN = 32 * NJ;
    static constexpr int KK = SB / 32;                       // 32-byte steps of a stage = shares of K
    static constexpr int NW = 4 / KK;                        // wavefronts side by side along N
    static constexpr int NJW = NJ / NW;                      // 32-column tiles of a wavefront
    static constexpr int NP = T::kPlanes;
    static constexpr int A_BYTES = BM * SB, B_BYTES = BN * SB;
    static constexpr int STAGE = A_BYTES + NP * B_BYTES;
    static constexpr int RED_BYTES = KK * BM * BN * 4;       // partial tiles of the epilogue
    static constexpr int RING_BYTES = NS * STAGE > RED_BYTES ? NS * STAGE : RED_BYTES;
    static constexpr int LDS_BYTES = RING_BYTES + OutSide<Store, BM>::BYTES;
    static_assert(SB == 64 || SB == 128, "stage rows of 64 or 128 bytes");
    static_assert(NJ % NW == 0 && NS >= 2, "tile shape");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
};

template <class T, int MI, int NJ, int SB, int NS, class Store>
__device__ __forceinline__ void slice_gemm_tile(const GemmArgs &g, const Store &store, int block, uint8_t *lds) {
    using S = SliceShape<T, MI, NJ, SB, NS, Store>;
    constexpr int CPR = SB / 16, RPI = 1024 / SB;            // 16-byte chunks per LDS row, LDS rows per direct load
    constexpr int A_TOT = S::BM / RPI, B_TOT = S::BN / RPI;  // direct loads per stage: A, one plane of B
    constexpr int A_INSTR = A_TOT < 4 ? 1 : A_TOT / 4;       // per wavefront (fewer than four: two wavefronts load the same rows)
    constexpr int B_INSTR = B_TOT < 4 ? 1 : B_TOT / 4;
    constexpr int LOADS = A_INSTR + S::NP * B_INSTR;
    static_assert((NS - 2) * LOADS < 64, "vmcnt is a 6-bit counter");
    typedef typename AccElem<T>::type elem_t;

    const int32_t *rows;
    long n_rows;
    resolve_rows(g.sel, rows, n_rows);
    // the same XCD-aware walk over the output as in nt_gemm_tile
    int row_tile, col_tile;
    g.tile_of(block, row_tile, col_tile);
    const long m0 = (long)row_tile * S::BM;
    if (m0 >= n_rows || col_tile >= g.col_tiles) return;
    const int n0 = col_tile * S::BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = g.N;
    const size_t row_bytes = (size_t)g.K * T::kElemBytes;
    const size_t a_row_bytes = (size_t)(g.a_ld > 0 ? g.a_ld : g.K) * T::kElemBytes;
    const int a_valid_bytes = (g.a_valid > 0 ? g.a_valid : g.K) * T::kElemBytes;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;

    // what each lane fetches (rows past the end are clamped to the last valid one: computed, never stored)
    const uint8_t *a_src[A_INSTR];
    const uint8_t *b_src[S::NP][B_INSTR];
    const int lr = lane / CPR, lc = lane % CPR;
#pragma unroll
    for (int i = 0; i < A_INSTR; ++i) {
        const int r = ((wave * A_INSTR + i) % A_TOT) * RPI + lr;
        long m = m0 + r;
        m = m < n_rows ? m : n_rows - 1;
        const long src = (g.gather_a && rows) ? (long)rows[m] : m;
        a_src[i] = static_cast<const uint8_t *>(g.a) + (size_t)src * a_row_bytes + swizzle<CPR>(r, lc) * 16;
    }
#pragma unroll
    for (int i = 0; i < B_INSTR; ++i) {
        const int r = ((wave * B_INSTR + i) % B_TOT) * RPI + lr;
        const int n = min(n0 + r, N - 1);
#pragma unroll
        for (int p = 0; p < S::NP; ++p)
            b_src[p][i] = static_cast<const uint8_t *>(g.b[p]) + (size_t)n * row_bytes + swizzle<CPR>(r, lc) * 16;
    }
    // 64-byte stages: rows of A may end inside the last stage (see nt_gemm_tile); the lane then re-reads their last 16 bytes
    const int a_klim = SB == 64 ? a_valid_bytes - 16 - swizzle<CPR>(lr, lc) * 16 : 0;

    auto issue_stage = [&](int slot_, int kbyte) {
        const uint32_t base = lds_base + slot_ * S::STAGE;
#pragma unroll
        for (int i = 0; i < A_INSTR; ++i)
            direct_load_16(a_src[i] + (SB == 64 ? min(kbyte, a_klim) : kbyte), base + ((wave * A_INSTR + i) % A_TOT) * 1024);
#pragma unroll
        for (int p = 0; p < S::NP; ++p)
#pragma unroll
            for (int i = 0; i < B_INSTR; ++i)
                direct_load_16(b_src[p][i] + kbyte, base + S::A_BYTES + p * S::B_BYTES + ((wave * B_INSTR + i) % B_TOT) * 1024);
    };

    typename T::Acc acc[MI][S::NJW];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < S::NJW; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    const int kk = wave % S::KK, wn = (wave / S::KK) * S::NJW * 32;
    const int fr = lane & 31, fg = lane >> 5;
    const int frag = fr * SB + swizzle<CPR>(fr, 2 * kk + fg) * 16;      // the swizzle depends on the row modulo 16 only

    const int n_stages = (int)(row_bytes / SB);
    const OutSide<Store, S::BM> side{store, rows, m0, n_rows, lds + S::RING_BYTES};
    side.fetch_rows(wave, lane);
#pragma unroll
    for (int q = 0; q < NS - 1; ++q)
        if (q < n_stages) issue_stage(q, q * SB);
    int slot_r = 0, slot_w = NS - 1;                          // ring slots of stage s and of stage s + NS - 1
    for (int s = 0; s < n_stages; ++s) {
        const int later = n_stages - 1 - s;                   // stages after s whose loads have been issued
        if (later >= NS - 2)
            wait_loads_in_flight<(NS - 2) * LOADS>();
        else
            static_for<NS - 2>([&](auto c) {
                constexpr int l = decltype(c)::value;
                if (later == l) wait_loads_in_flight<l * LOADS>();
            });
        __syncthreads();                                      // stage s is there; everyone has read stage s - 1
        if (s == 0) side.fetch_gates(wave, lane);
        if (s + NS - 1 < n_stages) issue_stage(slot_w, (s + NS - 1) * SB);
        const uint8_t *A = lds + slot_r * S::STAGE + frag, *B = lds + slot_r * S::STAGE + S::A_BYTES + wn * SB + frag;
        uint4 af[MI], bf[S::NP][S::NJW];
#pragma unroll
        for (int i = 0; i < MI; ++i) af[i] = *reinterpret_cast<const uint4 *>(A + i * 32 * SB);
#pragma unroll
        for (int p = 0; p < S::NP; ++p)
#pragma unroll
            for (int j = 0; j < S::NJW; ++j)
                bf[p][j] = *reinterpret_cast<const uint4 *>(B + p * S::B_BYTES + j * 32 * SB);
#pragma unroll
        for (int p = 0; p < S::NP; ++p)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < S::NJW; ++j) acc[i][j] = T::mma(af[i], bf[p][j], acc[i][j]);
        slot_r = slot_r + 1 == NS ? 0 : slot_r + 1;
        slot_w = slot_w + 1 == NS ? 0 : slot_w + 1;
    }

    // ---- where this lane's chunks go and what they need from memory: asked for before the partial tiles meet
    constexpr int ES = Store::kBytes, EPC = 16 / ES;          // elements of a 16-byte output chunk
    constexpr int CHUNK_ROWS = 256 / (S::BN / EPC), NC = (S::BM + CHUNK_ROWS - 1) / CHUNK_ROWS;
    const int nl = tid % (S::BN / EPC) * EPC, cr = tid / (S::BN / EPC);       // its first column, its first row
    const ChunkOut<Store> chunk(store, n0 + nl, N);
    wait_loads_in_flight<0>();
    float4 ext[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) ext[q] = chunk.fetch(side.dest(min(q * CHUNK_ROWS + cr, S::BM - 1)));

    // ---- the partial tiles meet in LDS
    elem_t *red = reinterpret_cast<elem_t *>(lds);
    const uint8_t *table = side.lds;
    constexpr int TILE = S::BM * S::BN;
    __syncthreads();                                          // the last stage has been read, `side` is complete
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < S::NJW; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                red[kk * TILE + (i * 32 + mfma32_row(r, lane)) * S::BN + wn + j * 32 + fr] = acc[i][j][r];
    __syncthreads();

    if constexpr (Store::kSignCodes) {
        if (n0 < store.code_cols) {                           // uniform: a 64-column tile is one code word of a head
            static_assert(S::BN == 64, "a tile must be one code word wide");
            const int part = n0 / store.part_width, cin = n0 - part * store.part_width;
            const int head = cin / store.head_dim, w = (cin % store.head_dim) / 64, W = store.head_dim / 64;
            uint64_t *dst = part == 0 ? store.codes[0] : store.codes[1];
            uint64_t mine = 0;
#pragma unroll
            for (int q = 0; q < S::BM / 4; ++q) {
                elem_t a = red[(wave * (S::BM / 4) + q) * S::BN + lane];
#pragma unroll
                for (int k = 1; k < S::KK; ++k) a += red[k * TILE + (wave * (S::BM / 4) + q) * S::BN + lane];
                const uint64_t word = __ballot(a >= 0);
                if (lane == q) mine = word;
            }
            const long m = m0 + wave * (S::BM / 4) + lane;
            if (lane < S::BM / 4 && m < n_rows) {
                const long b = m / store.tokens, n = m % store.tokens;
                dst[((size_t)(b * store.heads + head) * store.tokens + n) * W + w] = mine;
            }
            return;
        }
    }

#pragma unroll
    for (int q = 0; q < NC; ++q) {
        const int ml = q * CHUNK_ROWS + cr, n = n0 + nl;
        if (ml >= S::BM || m0 + ml >= n_rows || chunk.live <= 0) continue;
        uint32_t bits[EPC];
#pragma unroll
        for (int e4 = 0; e4 < EPC / 4; ++e4) {
            elem_t a[4];
#pragma unroll
            for (int k = 0; k < S::KK; ++k) {
                const uint4 t = *reinterpret_cast<const uint4 *>(red + k * TILE + ml * S::BN + nl + 4 * e4);
                const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const elem_t val = __builtin_bit_cast(elem_t, w[e]);
                    a[e] = k == 0 ? val : a[e] + val;
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) bits[4 * e4 + e] = store.convert(a[e], min(n + 4 * e4 + e, N - 1), table);
        }
        uint4 v;
        if constexpr (ES == 4)
            v = make_uint4(bits[0], bits[1], bits[2], bits[3]);
        else if constexpr (ES == 2)
            v = make_uint4(bits[0] | (bits[1] << 16), bits[2] | (bits[3] << 16), bits[4] | (bits[5] << 16), bits[6] | (bits[7] << 16));
        else {
            uint32_t w[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q] = bits[4 * q] | (bits[4 * q + 1] << 8) | (bits[4 * q + 2] << 16) | (bits[4 * q + 3] << 24);
            v = make_uint4(w[0], w[1], w[2], w[3]);
        }
        chunk.put(v, ext[q], side.gate(ml), side.dest(ml));
    }
}

template <class T, int MI, int NJ, int SB, int NS>
struct SliceTile {
    static constexpr int BM = 32 * MI, BN = 32 * NJ;
    template <class Store>
    static constexpr int lds_bytes() { return SliceShape<T, MI, NJ, SB, NS, Store>::LDS_BYTES; }
    template <class Store>
    __device__ static __forceinline__ void run(const GemmArgs &g, const Store &store, int block, uint8_t *lds) {
        slice_gemm_tile<T, MI, NJ, SB, NS, Store>(g, store, block, lds);
    }
    // A is fetched by col_groups L2s and each B plane by 8 / col_groups: the fewest bytes
    static int col_groups(const GemmArgs &g) {
        const long col_tiles = (g.N + BN - 1) / BN;
        const double a_bytes = (double)g.sel.max_rows * g.K * T::kElemBytes, b_bytes = (double)T::kPlanes * g.N * g.K * T::kElemBytes;
        int cg = 1;
        while (cg < 8 && 2 * cg <= col_tiles && a_bytes * 2 * cg + b_bytes * (4.0 / cg) < a_bytes * cg + b_bytes * (8.0 / cg)) cg *= 2;
        return cg;
    }
};

}  // namespace sa
