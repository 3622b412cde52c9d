// Hashing through the matrix cores, still bit-exact (Sec. 4.1, binary quantisation of Q / K).
//
// The code bit is DEFINED as the sign of the fp32 chain acc = fma(x_k, r_kj, acc), k ascending.
// For almost every (row, bit) that sign is decided long before rounding matters, so the kernel
//   1. computes z~ = x . r^_j on the fp16 matrix cores, r^_j = r_j / |r_j|, with a three-product split
//      (x = xh + xl, r^ = rh + rl, each fp16 rounded to nearest; z~ = xh rh + xh rl + xl rh),
//   2. keeps sign(z~) wherever |z~| > theta |x|.  theta is 2^-16, 2^-15 and 2^-14 at d = 32, 64 and 128; hash_margin.h adds up
//      what it has to cover (1.49, 2.87 and 5.60 e-5 against 1.53, 3.05 and 6.10 e-5), and
//   3. re-runs the defining chain, one (row, bit) per lane, for the rest (0.02 % of the bits on Gaussian data at
//      d = 64; every bit if the data is degenerate) and flips the stored bit if needed.
// NaN / Inf / denormal-range sums fail the test in step 2 and take step 3, which is the definition.
//
// A wavefront takes tiles of 32 consecutive rows of the flattened [B*N*H, d] input as two units of 16.  The MFMA
// (16x16x32) computes the TRANSPOSED tile, hash columns down and rows across; the columns are dealt to its rows so that a
// lane ends up with a quarter of the code bits of one row, consecutive ones.  The hash matrix lives in LDS, as ready-made
// fragments and as fp32 columns for step 3; the rows of the next tile are in flight while a tile is multiplied.
//
// A load instruction takes 32 bytes of each of the 32 rows, so that its first use of a line asks for all rows' lines at
// once; the operands, which want 64 bytes of 16 rows, are put together by lane swaps after the split.  Loaded as 64 bytes of
// 16 rows, the attention of 32 x 3136 tokens x 1 head x 32 with 64 bits takes 25.2 us (24.5 now).
// At 256 columns rows that fill the memory-side cache (256 MiB) by themselves are loaded as a stream: the products hide most of it,
// and V, which K^T V reads next, stays there (block of 8 x 16384 tokens x 4 heads, 256 MiB of Q and K, 382.1 -> 378.1 us, of 6 x
// 16384 348.5 -> 345.2; without the MLP 215.5 -> 218.5).  Fewer are still there from whoever wrote them, or from the last pass: blocks
// of 4 x 16384 tokens, 128 MiB, 199.5 us, as a stream 210.7; of 64 x 197 x 12 heads, 73 MiB, 200.8 and 206.6; the hash of those
// alone 34.0 and 39.1.  At 64 columns the wait shows (24.5 -> 28.4).
// Products of 32x32x16 took the same time here but more power, which the kernels around it paid for in clock.
//
// What bounds it: at 256 bits the products and the vector work in their shadow (16 funnel shifts and 8 three-way minima
// per 16 bits, 7 operations to split two elements); at 128 bits and fewer the rows of Q and K, with about 4.5 us before the
// first product (3.5 of them the launch, 1 until the hash matrix has arrived) and 1 us of re-runs at the end.  At d = 64 and 128 more
// wavefronts or rows in flight gave nothing there.  The fragments are made from the registers the hash matrix is loaded
// into: through LDS, with two more barriers and two passes over its fp32 form, a launch took 0.8 us longer at d = 64 and up
// to 3.7 at d = 128.  Q and K, alone and over and over, 64 bytes of 16 rows per load -> now:
//   64 x 197 x 12 heads x 64 -> 128 bits  25.1 -> 23.6 us      64 x 197 x 12 x 64 -> 64  19.2 -> 18.6
//   64 x 197 x 3 x 64 -> 64               10.0 ->  9.2          8 x 1000 x 3 x 128 -> 128  14.8 -> 14.7
//   32 x 3136 x 1 x 32 -> 64              11.0 -> 10.3 (8.1 by launch_waves)   1 x 197 x 3 x 64 -> 64      5.8 ->  5.7
//    1 x 16384 x 4 x 64 -> 256            18.5 -> 17.4          8 x 16384 x 4 x 64 -> 256  110 -> 112 (as a stream; 104 without)
#include "common.h"
#include "hash_tile.h"
#include "side_work.h"

namespace sa {

namespace {

constexpr int kListCap = 128;                 // unsettled bits parked per wavefront

// Swaps a's upper 32 lanes with b's lower 32.
template <typename T>
__device__ inline void swap_halves(T &a, T &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    a = __builtin_bit_cast(T, r0);
    b = __builtin_bit_cast(T, r1);
}

// D: head dim; C: hash columns of a workgroup (blockIdx.y selects the group); kWaves: its wavefronts.
template <int D, int C, int kWaves, bool STREAM>
__global__ __launch_bounds__(kWaves * 64) void binarize_mfma_kernel(Tensors ts, const float *__restrict__ proj, uint32_t rows,
                                                                    RowMap map, int nbits, uint32_t n_tiles, uint32_t n_total,
                                                                    uint32_t hash_blocks, SideWork side) {
    constexpr int S = D / 32;                     // MFMA steps along k
    constexpr int T = C / 16;                     // 16-column tiles
    constexpr int GROUPS = T / 4;                 // of four tiles: 16 bits of a lane
    constexpr int L4 = D / 8;                     // 16-byte loads per lane
    constexpr int THREADS = kWaves * 64;
    constexpr int BYTES = C / 32;                 // code bytes of a lane: columns (C / 4) g .. of its row
    __shared__ __attribute__((aligned(16))) uint4 frag_s[T * S * 2 * 64];       // [tile][step][upper, lower][lane]
    __shared__ __attribute__((aligned(16))) float r_s[D * C];
    // hash matrix: a task is eight k of one column, four tasks per 32 k; a thread's tasks are of one column
    constexpr int TPC = THREADS / C < 4 * S ? THREADS / C : 4 * S;         // threads that share a column
    constexpr int TASKS = 4 * S / TPC;
    static_assert(THREADS % C == 0 && TASKS * TPC == 4 * S, "the threads of a column share its tasks evenly");
    __shared__ float n2_s[TPC][C];
    __shared__ uint64_t list_s[kWaves][kListCap];
    __shared__ int cnt_s[kWaves];

    if (blockIdx.x >= hash_blocks) {
        side_block<kWaves * 64>(side, (long)(blockIdx.x - hash_blocks) * gridDim.y + blockIdx.y);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int c_first = blockIdx.y * C;

    // row 16 (g / 2) + n of a tile: its lane loads k = 8 j + 4 (g % 2) .. + 3, j = 0 .. L4 - 1.  Tiles 0 .. n_tiles - 1
    // belong to the first tensor, the next n_tiles to the second; rows past the end re-read the last one.
    v4f xn[L4];
    auto load_tile = [&](uint32_t tile) {
        const bool second = tile >= n_tiles;
        const float *x = second ? ts.x1 : ts.x0;
        const uint32_t r0 = (second ? tile - n_tiles : tile) * 32;
        const float *xr = x + (size_t)min(r0 + 16 * (g >> 1) + n, rows - 1) * D + 4 * (g & 1);
#pragma unroll
        for (int j = 0; j < L4; ++j) {
            const v4f *at = reinterpret_cast<const v4f *>(xr + 8 * j);
            xn[j] = STREAM ? __builtin_nontemporal_load(at) : *at;
        }
    };
    const uint32_t tile_step = hash_blocks * kWaves;
    uint32_t tile = blockIdx.x * kWaves + wave;

    // ---- hash matrix: fp32 columns to LDS for step 3, their norms, then the fragments of the normalised columns, from the
    //      registers the columns came in.  Asked for before the first rows, which then need not have arrived.
    {
        const int c = tid % C, part = tid / C;
        const int q = c / (C / 4), w = c % (C / 4);               // lane group of the accumulator, bit within it
        const int t = w / 4, rho = 4 * q + w % 4;                 // tile and its row
        const bool mine = part < TPC;
        float v[TASKS][8];
        auto k_of = [&](int i, int e) {
            const int j = part + i * TPC;                         // task j: s = j / 4, kq = j % 4
            return 32 * (j >> 2) + 16 * (e / 4) + 4 * (j & 3) + e % 4;
        };
        if (mine) {
#pragma unroll
            for (int i = 0; i < TASKS; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[i][e] = proj[(size_t)k_of(i, e) * nbits + c_first + c];
        }
        if (tile < n_total) load_tile(tile);
        if (mine) {
            float n2 = 0.0f;                                      // this thread's share of the norm
#pragma unroll
            for (int i = 0; i < TASKS; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    r_s[k_of(i, e) * C + c] = v[i][e];
                    n2 = __builtin_fmaf(v[i][e], v[i][e], n2);
                }
            n2_s[part][c] = n2;
        }
        __syncthreads();
        if (mine) {
            float n2 = 0.0f;
#pragma unroll
            for (int p = 0; p < TPC; ++p) n2 += n2_s[p][c];
            // a dead, denormal, overflowing or non-finite column gets an all-zero r^: z~ = 0 fails the margin test, so
            // every bit of that column is parked and settled by the defining chain
            const float inv = n2 >= kColumnMin2 && n2 < __builtin_inff() ? 1.0f / __builtin_sqrtf(n2) : 0.0f;
#pragma unroll
            for (int i = 0; i < TASKS; ++i) {
                const int j = part + i * TPC, step = j >> 2, kq = j & 3;
                uint32_t up[4], lo[4];
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2) {
                    float x[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) x[h] = inv > 0.0f ? v[i][2 * e2 + h] * inv * kColumnScale : 0.0f;
                    split_f16_pair(x[0], x[1], up[e2], lo[e2]);
                }
                frag_s[((t * S + step) * 2 + 0) * 64 + kq * 16 + rho] = make_uint4(up[0], up[1], up[2], up[3]);
                frag_s[((t * S + step) * 2 + 1) * 64 + kq * 16 + rho] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            }
        }
        __syncthreads();
    }

    int cnt = 0;                   // parked entries of this wavefront (wave-uniform)
    uint64_t *list = list_s[wave];
    auto work_off = [&]() {
        wait_loads_in_flight<0>();               // the words these bits live in have been stored
#pragma unroll 1
        for (int t0 = 0; t0 < cnt; t0 += 64)
            if (t0 + lane < cnt) settle_entry<D, 16>(list[t0 + lane], ts, r_s, C, c_first, map);
        cnt = 0;
    };

    for (; tile < n_total; tile += tile_step) {
        const bool second = tile >= n_tiles;
        const uint32_t r0 = (second ? tile - n_tiles : tile) * 32;
        uint8_t *codes = reinterpret_cast<uint8_t *>(second ? ts.codes1 : ts.codes0);

        // |x_row|^2: keep sign(z~) where |z~| > keep (in units of the staged columns); a non-finite |x|^2 keeps nothing
        float nx2 = 0.0f;
#pragma unroll
        for (int j = 0; j < L4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) nx2 = __builtin_fmaf(xn[j][i], xn[j][i], nx2);
        nx2 += __shfl_xor(nx2, 16);
        // Rows of ordinary magnitude (|x| in 2^-2 .. 2^12) split as they are, others are brought to |x| ~ 1 first (hash_margin.h).
        float unit = 1.0f;
        if (__ballot(!(nx2 >= kOrdinaryMin2 && nx2 <= kOrdinaryMax2)) != 0) {          // wave-uniform
            int e = 0;
            if (nx2 > 0.0f && nx2 < __builtin_inff()) e = __builtin_amdgcn_frexp_expf(nx2) / 2;
            unit = __builtin_amdgcn_ldexpf(1.0f, -e);
#pragma unroll
            for (int j = 0; j < L4; ++j) xn[j] *= unit;
        }
        const float kept = nx2 < __builtin_inff()
                               ? __builtin_fmaxf(hash_theta(D) * __builtin_sqrtf(nx2), kKeepFloor) * unit * kColumnScale
                               : __builtin_inff();
        float keep[2] = {kept, kept};              // of rows n and 16 + n
        swap_halves(keep[0], keep[1]);
        // Operands: of two loads side by side the second's lower lanes and the first's upper ones change places: then a lane
        // has its four of both loads' 16 k of row n in one and of row 16 + n in the other.
        v8h xh[2][S], xl[2][S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            uint32_t up[2][4], lo[2][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const v4f v = xn[4 * s + j];
                split_f16_pair(v[0], v[1], up[j & 1][2 * (j >> 1)], lo[j & 1][2 * (j >> 1)]);
                split_f16_pair(v[2], v[3], up[j & 1][2 * (j >> 1) + 1], lo[j & 1][2 * (j >> 1) + 1]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                swap_halves(up[0][i], up[1][i]);
                swap_halves(lo[0][i], lo[1][i]);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                xh[u][s] = __builtin_bit_cast(v8h, make_uint4(up[u][0], up[u][1], up[u][2], up[u][3]));
                xl[u][s] = __builtin_bit_cast(v8h, make_uint4(lo[u][0], lo[u][1], lo[u][2], lo[u][3]));
            }
        }
        if (tile + tile_step < n_total) load_tile(tile + tile_step);

        // 16 bits of every lane (a group of four tiles) at a time; accumulator register r of tile t: bit 4 t + r of the
        // lane's quarter.  The products of a group are issued with the signs and minima of the group before it between
        // them (the wavefront issues in order: behind the products the vector work would wait for all of them), and
        // the fragments of a step are read one step ahead.
        constexpr int ITEMS = S * 4;                               // (step, tile) of a group
        uint32_t word[2][(GROUPS + 1) / 2], park[2][(GROUPS + 1) / 2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < (GROUPS + 1) / 2; ++q) word[u][q] = park[u][q] = 0;
        v4f acc[2][2][4];                                          // [group parity][unit][tile]
        v8h fr[2][2];                                              // [parity][upper, lower]
        auto read_item = [&](int grp, int item, v8h (&f)[2]) {
            const uint4 *at = frag_s + (((grp * 4 + item % 4) * S + item / 4) * 2) * 64 + lane;
            f[0] = __builtin_bit_cast(v8h, at[0]);
            f[1] = __builtin_bit_cast(v8h, at[64]);
        };
        auto multiply_group = [&](int grp) {
            v4f (&a)[2][4] = acc[grp & 1];
#pragma unroll
            for (int item = 0; item < ITEMS; ++item) {
                const int s = item / 4, t = item % 4;
                const v8h rh = fr[item & 1][0], rl = fr[item & 1][1];
                if (item + 1 < ITEMS) read_item(grp, item + 1, fr[(item + 1) & 1]);
                else if (grp + 1 < GROUPS) read_item(grp + 1, 0, fr[(item + 1) & 1]);
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    a[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(rh, xh[u][s], s == 0 ? v4f{0.0f, 0.0f, 0.0f, 0.0f} : a[u][t], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 2; ++u) a[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(rl, xh[u][s], a[u][t], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 2; ++u) a[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(rh, xl[u][s], a[u][t], 0, 0, 0);
            }
        };
        static_assert(ITEMS % 2 == 0, "the fragment buffers alternate across groups");
        read_item(0, 0, fr[0]);
        multiply_group(0);
#pragma unroll
        for (int grp = 0; grp < GROUPS; ++grp) {
            __builtin_amdgcn_sched_barrier(0);
            if (grp + 1 < GROUPS) multiply_group(grp + 1);
            float smallest[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const v4f (&z)[4] = acc[grp & 1][u];
                uint32_t neg = 0;                                  // bit q = sign of element q (-0 is parked anyway)
                smallest[u] = __builtin_inff();
#pragma unroll
                for (int q = 15; q >= 0; --q) {
                    const float zq = z[q / 4][q % 4];
                    neg = __builtin_amdgcn_alignbit(neg, __builtin_bit_cast(uint32_t, zq), 31);
                    smallest[u] = __builtin_fminf(smallest[u], __builtin_fabsf(zq));
                }
                word[u][grp / 2] |= (~neg & 0xFFFFu) << (16 * (grp & 1));
            }
            if (grp + 1 < GROUPS) {
#pragma unroll
                for (int item = 0; item < ITEMS; ++item) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);             // the next fragments
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);         // a product
                        __builtin_amdgcn_sched_group_barrier(0x002, ITEMS == 4 ? 3 : 2, 0);    // what its shadow holds
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(word[u][grp / 2]));      // now, not behind the last group's products
            // the smallest |z~| of the 16 decides for all of them; only where one is in doubt they are looked at
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (__ballot(!(smallest[u] > keep[u])) != 0) {     // wave-uniform
                    uint32_t pk = 0;
#pragma unroll
                    for (int q = 0; q < 16; ++q)
                        pk |= (uint32_t)(!(__builtin_fabsf(acc[grp & 1][u][q / 4][q % 4]) > keep[u])) << q;
                    park[u][grp / 2] |= pk << (16 * (grp & 1));
                }
        }

        uint32_t any_park = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t row = r0 + 16 * u + n;
            const bool row_ok = row < rows;
            uint8_t *dst = codes + map.row_words(min(row, rows - 1)) * 8 + c_first / 8 + BYTES * g;
            if (row_ok) {
                if constexpr (BYTES == 2) *reinterpret_cast<uint16_t *>(dst) = (uint16_t)word[u][0];
                else if constexpr (BYTES == 4) *reinterpret_cast<uint32_t *>(dst) = word[u][0];
                else *reinterpret_cast<uint2 *>(dst) = make_uint2(word[u][0], word[u][GROUPS / 2 - 1]);
            }
#pragma unroll
            for (int q = 0; q < (GROUPS + 1) / 2; ++q) {
                if (!row_ok) park[u][q] = 0;
                any_park |= park[u][q];
            }
        }

        // park the unsettled bits.  The list may be worked off at any point from here on: this tile's words are on their
        // way to memory.
        while (__ballot(any_park != 0) != 0) {                    // wave-uniform; rarely more than 2 rounds
            constexpr int PIECES = 2 * ((GROUPS + 1) / 2);
            int which = 0;
            uint32_t mine = 0, bits = 0;                          // this lane's first non-empty piece
#pragma unroll
            for (int p = PIECES - 1; p >= 0; --p) {
                const uint32_t pk = park[p / (PIECES / 2)][p % (PIECES / 2)];
                if (pk) { which = p; mine = pk; bits = word[p / (PIECES / 2)][p % (PIECES / 2)]; }
            }
            const bool parked = any_park != 0;
            const int pos = parked ? __builtin_ctz(mine) : 0;
            const uint64_t pm = __ballot(parked);
            if (cnt + 64 > kListCap) work_off();
            if (parked) {
                const int slot = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(pm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pm, 0u));
                const int u = which / (PIECES / 2), piece = which % (PIECES / 2);
                list[slot] = open_bit(r0 + 16 * u + n, c_first + (C / 4) * g + 32 * piece + pos, (bits >> pos) & 1u, second);
                any_park = 0;
#pragma unroll
                for (int p = 0; p < PIECES; ++p) {
                    uint32_t &pk = park[p / (PIECES / 2)][p % (PIECES / 2)];
                    pk = p == which ? pk & (pk - 1u) : pk;
                    any_park |= pk;
                }
            }
            cnt += __builtin_popcountll(pm);
        }
    }

    // The wavefronts' leftovers are pooled and worked off 64 entries per pass, pass p by wavefront p % kWaves: the
    // cost of a pass is the latency of its loads, so full passes side by side beat nearly empty ones.
    wait_loads_in_flight<0>();                   // this wavefront's words have been stored
    if (lane == 0) cnt_s[wave] = cnt;
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) total += cnt_s[w];
    for (int t0 = wave * 64; t0 < total; t0 += THREADS) {
        int t = t0 + lane, w = 0;
        if (t < total) {
            while (t >= cnt_s[w]) t -= cnt_s[w++];
            settle_entry<D, D <= 64 ? D : 32>(list_s[w][t], ts, r_s, C, c_first, map);   // the tile loop's registers are free now
        }
    }
}

}  // namespace

bool binarize_mfma_supported(int d, int nbits) {
    return (d == 32 || d == 64 || d == 128) && nbits % 64 == 0;
}

template <int D, int C, int kWaves>
int launch_waves(const Tensors &ts, const float *proj, long rows, const RowMap &map, int nbits, long n_tiles, long n_total,
                 const SideWork &side, hipStream_t st) {
    // Eight wavefronts per CU (what the registers allow) over all column groups, every wavefront the same number of tiles.  At d = 32 and
    // 64 columns, whose tiles are short and little but their loads, sixteen, each of which takes what there is: 6272 tiles were four each
    // for 1568 wavefronts, with eight on one SIMD of two CUs and four on the next (Q and K of 32 x 3136 tokens x 32 with the Add
    // products 24.7 -> 22.9 us; 200704 rows alone 9.5 -> 8.1, 302592 11.9 -> 10.7, 2097152 61.4 -> 50.7; with twelve 11.2 and 52.5, with 24 12.1 and 52.3).
    // Longer tiles lose by it (d = 64: 302592 rows 18.0, 20.6; 128 bits 23.4, 28.1), and so does a launch that also routes, by its tail: its
    // last workgroups look at all tokens and wait for a place beside the sixteen (blocks with two experts, us with sixteen and eight:
    // 35 x 567 tokens x 2 heads 42.4, 41.6; x 4 heads 68.6, 66.2; 1 x 19845 x 2 46.0, 45.0; with places left free for them 42.5, 67.2, 46.4).
    // The decode of packed weights may ride along: it looks at nothing but its own share and only fills CUs that are done (blocks with a
    // Shift MLP on packed weights, us with eight and sixteen: 25088 tokens x 4 heads, 512 hidden 35.4, 33.6; 50176 x 2, 256 hidden 32.8,
    // 31.1; 12544 x 8, 1024 hidden 42.4, 40.9; the same up to 6272 tokens).
    constexpr bool SHORT = D == 32 && C == 64;
    const bool sixteen = SHORT && side.route.T == 0;
    const int per_cu = C != 64 ? 1 : (sixteen ? 16 : 8) / kWaves;
    const long waves = 256 * per_cu / (nbits / C) * kWaves;
    const long tiles_per_wave = sixteen ? 1 : (n_total + waves - 1) / waves;
    const long enough = (n_total + kWaves * tiles_per_wave - 1) / (kWaves * tiles_per_wave);
    const long blocks = enough < waves / kWaves ? enough : waves / kWaves;
    // what rides along comes behind the tiles: it fills the CUs that are done first
    const long more = (side_blocks<kWaves * 64>(side) + nbits / C - 1) / (nbits / C);
    const dim3 grid((unsigned)(blocks + more), (unsigned)(nbits / C));
    const bool stream = C == 256 && n_total * 32 * D * 4 >= (192L << 20);       // see the top
#define SA_HASH(STREAM_)                                                                                                          \
    binarize_mfma_kernel<D, C, kWaves, STREAM_><<<grid, dim3(kWaves * 64), 0, st>>>(                                              \
        ts, proj, (uint32_t)rows, map, nbits, (uint32_t)n_tiles, (uint32_t)n_total, (uint32_t)blocks, side)
    if (stream) SA_HASH(C == 256);
    else SA_HASH(false);
#undef SA_HASH
    return check_launch("sa_binarize(mfma)");
}

// Workgroups of 8 wavefronts, of 4 where those already have one tile each: two wavefronts of one tile on a SIMD only
// take turns (1 x 197 x 3 heads x 64 -> 64 bits: 7.6 -> 7.0 us).  64 columns take little LDS: two workgroups of 4 to a CU, each
// of which waits for fewer wavefronts (8 x 1000 x 3 heads x 128 -> 64 bits: 12.1 -> 11.5 us, 16 x 784 x 2 x 32 -> 64 5.8 -> 5.6).
// Unless they also route: a workgroup of 4 takes in 4096 tokens per round trip, and all of them look at all tokens (block of
// 32 x 784 tokens x 2 heads: 47.3 us with 4 wavefronts, 44.6 with 8).
template <int D, int C>
int launch_one(const Tensors &ts, int count, const float *proj, long rows, int N, int H, int nbits, const SideWork &side,
               hipStream_t st) {
    const long n_tiles = (rows + 31) / 32, n_total = n_tiles * count;
    const RowMap map{FastDiv((uint32_t)H), FastDiv((uint32_t)N), N, H, nbits / 64};
    const bool four = n_total <= 256 / (nbits / C) * 4 || (C == 64 && side.route.T <= 4096);
    return four ? launch_waves<D, C, 4>(ts, proj, rows, map, nbits, n_tiles, n_total, side, st)
                : launch_waves<D, C, 8>(ts, proj, rows, map, nbits, n_tiles, n_total, side, st);
}

// x1 / codes1 may be null: one tensor.  Columns of a workgroup: as many of the code as divide it, up to 256 (128 at
// d = 128: what the LDS holds), so that the rows are read and split as few times as possible.  But fewer while that leaves half
// of the chip's SIMDs without a tile: the time is then that of one tile and of its share of the hash matrix (Q and K of 1 x 197 x 3
// heads x 64 -> 256 bits 8.4 -> 5.8 us, -> 128 bits 6.9 -> 5.7, 4 x 137 x 12 x 64 -> 256 8.8 -> 7.3, 1 x 197 x 3 x 128 -> 128 10.4 ->
// 8.2; from 512 to 1024 tiles it is a tie, beyond slower: 4 x 1000 x 4 x 64 -> 256 8.9 against 10.3).
int launch_binarize_mfma(const float *x0, const float *x1, const float *proj, uint64_t *codes0, uint64_t *codes1,
                         long rows, int N, int H, int d, int nbits, hipStream_t st, const SideWork &side) {
    const Tensors ts{x0, x1, codes0, codes1};
    const int count = x1 ? 2 : 1;
    const long n_total = (rows + 31) / 32 * count;
    auto takes = [&](int c) { return nbits % c == 0 && n_total * (nbits / c) > 512; };
    const bool c128 = takes(128), c256 = takes(256);
    switch (d) {
        case 32:
            return c256   ? launch_one<32, 256>(ts, count, proj, rows, N, H, nbits, side, st)
                   : c128 ? launch_one<32, 128>(ts, count, proj, rows, N, H, nbits, side, st)
                          : launch_one<32, 64>(ts, count, proj, rows, N, H, nbits, side, st);
        case 64:
            return c256   ? launch_one<64, 256>(ts, count, proj, rows, N, H, nbits, side, st)
                   : c128 ? launch_one<64, 128>(ts, count, proj, rows, N, H, nbits, side, st)
                          : launch_one<64, 64>(ts, count, proj, rows, N, H, nbits, side, st);
        default:
            return c128 ? launch_one<128, 128>(ts, count, proj, rows, N, H, nbits, side, st)
                        : launch_one<128, 64>(ts, count, proj, rows, N, H, nbits, side, st);
    }
}

}  // namespace sa
