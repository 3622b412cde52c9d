// The Q, K, V projection of a layer and the hash of Q and K in one launch, for heads of 64 or 32 columns and rows that are too wide for a
// workgroup to hold or too many for norm_hash.hip:
//     (q, k, v)[row] = scale * Wqkv . codes[row],     bit j of q's code = [q[row, head] . proj[:, j] >= 0], k's alike
// The tiles are those of gemm_mfma.h, computed transposed: a wavefront has all columns of one or two heads for its rows, a lane half of one row's,
// which as fp16 terms are an operand of the hash's products as they stand (the k index of a product may be any permutation of the head's
// columns that both operands use).  The bits are kept or left to the defining chain as in binarize_mfma.hip; Q and K reach memory as code
// words and, for the chain, as the few rows with bits that the margin leaves open; V leaves as fp32.
//
// Saves the hash's launch and Q's and K's way through memory: layer of 12608 rows of 768, 128 bits 319 -> 303 us (in a trace 67; 57 + 27 as two).
// Bound by what a tile does behind its sums while the matrix cores have only this: the hash matrix's fragments, made by every workgroup
// from the columns in L2 (about 1.5 us), three products for every step, signs, and the chain's round trip to memory (with no open bits
// 3.5 us less).  Fragments are read a step ahead of their products: with the reads where they are used a 12608 x 768 layer took 10 us
// more.  Two column groups side by side gained nothing over that.
#include "common.h"
#include "gemm_common.h"
#include "gemm_mfma.h"
#include "gemm_stores.h"
#include "hash_tile.h"

namespace {

using namespace sa;

constexpr int kList = 96;                                    // open bits of a wavefront

// D: head width, 64 or 32 (a wavefront then has two heads).  NB: code bits.
template <int D, int NB>
struct HashStore : ShiftStore<kEpiQkvCodes> {
    static constexpr int GROUPS = NB / 32, STEPS = D / 16;   // of a product's columns, and of its sum
    static constexpr int TPC = 256 / NB, TASKS = D / 8 / TPC;              // threads of a hash column, eight rows of it for each task
    static_assert(D / 8 % TPC == 0 && (D == 64 || D == 32), "a hash column, once");
    static constexpr int FRAGS = 0, NORMS = NB * D * 4, LISTS = NORMS + 256 * 4, MASKS = LISTS + 4 * kList * 8;
    static constexpr int kHashBytes = MASKS + 2 * NB / 8;
    const float *proj;                   // [D, NB]
    Tensors of;                          // Q and K (rows with open bits), and where their codes go
    RowMap map;
    HashStore(const Epilogue &e, const float *p, const Tensors &t, const RowMap &m) : ShiftStore(e), proj(p), of(t), map(m) {}

    // acc: 32 MI rows from m on by the 64 columns from `col` on.  The stage buffers are free behind a barrier.
    template <int MI>
    __device__ __forceinline__ void hash(const v16i_t (&acc)[MI][2], uint8_t *lds, long m, long n_rows, int col, int tid) const {
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), fr = lane & 31, fg = lane >> 5;
        // ---- the hash matrix, as fragments of its normalised columns (upper and lower fp16 terms).  Half f of a wavefront gets the
        //      columns NB / 2 f .. of a product's result, 16 of each group.
        const int hc = tid % NB, part = tid / NB;
        auto k_of = [&](int i, int e) {                      // task j: what lanes 32 (j & 1) .. hold of step j / 2
            const int j = part + i * TPC;
            return 16 * (j >> 1) + 8 * (e / 4) + 4 * (j & 1) + e % 4;
        };
        float hv[TASKS][8], n2 = 0.0f;
#pragma unroll
        for (int i = 0; i < TASKS; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) hv[i][e] = proj[(size_t)k_of(i, e) * NB + hc];
#pragma unroll
        for (int i = 0; i < TASKS; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) n2 = __builtin_fmaf(hv[i][e], hv[i][e], n2);
        wait_loads_in_flight<0>();
        __syncthreads();                                     // the last stage has been read
        float *norms = reinterpret_cast<float *>(lds + NORMS);
        norms[part * NB + hc] = column_norm(n2, hv);
        __syncthreads();
        uint4 *frags = reinterpret_cast<uint4 *>(lds + FRAGS);
        uint64_t *zero_columns = reinterpret_cast<uint64_t *>(lds + MASKS), *unbounded_columns = zero_columns + NB / 64;     // bit: a column
        {
            n2 = 0.0f;
#pragma unroll
            for (int p = 0; p < TPC; ++p) n2 += norms[p * NB + hc];
            const uint64_t zero = __ballot(n2 == 0.0f), unbounded = __ballot(!(n2 < __builtin_inff()));
            if (part == 0 && lane == 0) {
                zero_columns[hc / 64] = zero;
                unbounded_columns[hc / 64] = unbounded;
            }
            // a column of no use (see binarize_mfma.hip) is left to the chain, unless it is all zeros
            const float inv = n2 >= kColumnMin2 && n2 < __builtin_inff() ? 1.0f / __builtin_sqrtf(n2) : 0.0f;
            const int f = hc / (NB / 2), c = hc % (NB / 2), rho = 8 * (c % 16 / 4) + 4 * f + c % 4;
#pragma unroll
            for (int i = 0; i < TASKS; ++i) {
                const int j = part + i * TPC;
                uint32_t up[4], lo[4];
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2) {
                    float x[2];
#pragma unroll
                    for (int o = 0; o < 2; ++o) x[o] = inv > 0.0f ? hv[i][2 * e2 + o] * inv * kColumnScale : 0.0f;
                    split_f16_pair(x[0], x[1], up[e2], lo[e2]);
                }
                uint4 *at = frags + ((c / 16 * STEPS + (j >> 1)) * 2) * 64 + (j & 1) * 32 + rho;
                at[0] = make_uint4(up[0], up[1], up[2], up[3]);
                at[64] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            }
        }
        __syncthreads();

        uint32_t some_zeros = 0;
#pragma unroll
        for (int q = 0; q < NB / 32; ++q) some_zeros |= reinterpret_cast<const uint32_t *>(zero_columns)[q];
        const bool any_zeros = __builtin_amdgcn_readfirstlane(some_zeros) != 0;
        uint64_t *list = reinterpret_cast<uint64_t *>(lds + LISTS) + wave * kList;
        int cnt = 0;                                         // entries of it (wave-uniform)
        auto work_off = [&](auto steps_c) {                  // steps of the chain whose operands are loaded at once
            if (cnt == 0) return;
            wait_loads_in_flight<0>();                       // the words these bits live in and the rows have been stored
#pragma unroll 1
            for (int t0 = 0; t0 < cnt; t0 += 64)
                if (t0 + lane < cnt) settle_entry<D, decltype(steps_c)::value>(list[t0 + lane], of, proj, NB, 0, map);
            cnt = 0;
        };
        const bool second = col >= part_width;
        const int in_part = second ? col - part_width : col, head0 = in_part / D;
        float *rows = const_cast<float *>(second ? of.x1 : of.x0) + in_part;
        uint64_t *codes = second ? of.codes1 : of.codes0;
        static_for<MI * (64 / D)>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value / (64 / D), of_pair = decltype(i_c)::value % (64 / D);
            const int head = head0 + of_pair;
            const long row = m + 32 * i + fr;
            const bool valid = row < n_rows;
            auto value = [&](int j, int r) { return __builtin_fmaf((float)acc[i][of_pair + j][r], scale, 0.0f); };
            float nx2 = 0.0f;
#pragma unroll
            for (int j = 0; j < D / 32; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) nx2 = __builtin_fmaf(value(j, r), value(j, r), nx2);
            nx2 += __shfl_xor(nx2, 32);
            // rows of ordinary magnitude split as they are, others are brought to |x| ~ 1 first (hash_margin.h)
            v8h xh[STEPS], xl[STEPS];
            auto split = [&](float unit) {
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    uint32_t up[4], lo[4];
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2)
                        split_f16_pair(value(s >> 1, 8 * (s & 1) + 2 * e2) * unit, value(s >> 1, 8 * (s & 1) + 2 * e2 + 1) * unit, up[e2], lo[e2]);
                    xh[s] = __builtin_bit_cast(v8h, make_uint4(up[0], up[1], up[2], up[3]));
                    xl[s] = __builtin_bit_cast(v8h, make_uint4(lo[0], lo[1], lo[2], lo[3]));
                }
            };
            float unit = 1.0f;
            bool zero = false;                               // a row of zeros: hash_tile.h
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
            const uint32_t t = (uint32_t)min(row, n_rows - 1), b = map.by_n(t), n = t - b * (uint32_t)map.N;
            uint8_t *word = reinterpret_cast<uint8_t *>(codes + (((size_t)b * map.H + head) * map.N + n) * (NB / 64)) + NB / 16 * fg;
            // fragments of step STEPS g + s, one step ahead of their products
            uint4 part_of[2][2];
            auto read = [&](int step, uint4 (&to)[2]) {
                to[0] = frags[step * 128 + lane];
                to[1] = frags[step * 128 + 64 + lane];
            };
            read(0, part_of[0]);
#pragma unroll 1
            for (int g = 0; g < GROUPS; ++g) {
                const int bit0 = NB / 2 * fg + 16 * g;
                v16f_t z;
#pragma unroll
                for (int q = 0; q < 16; ++q) z[q] = 0.0f;
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    read(min(STEPS * g + s + 1, STEPS * GROUPS - 1), part_of[(s + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int term = 0; term < 3; ++term)             // xh rh, xh rl, xl rh
                        z = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, part_of[s & 1][term == 1]), term == 2 ? xl[s] : xh[s], z, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                uint32_t neg = 0;                            // bit q: sign of element q (-0 is open anyway)
                float smallest = __builtin_inff();
#pragma unroll
                for (int q = 15; q >= 0; --q) {
                    const float zq = z[q];                   // (a bit cast of z[q] itself takes z[0])
                    neg = __builtin_amdgcn_alignbit(neg, __builtin_bit_cast(uint32_t, zq), 31);
                    smallest = __builtin_fminf(smallest, __builtin_fabsf(zq));
                }
                const uint32_t bits = ~neg & 0xffffu;
                if (valid) *reinterpret_cast<uint16_t *>(word + 2 * g) = (uint16_t)bits;
                if (__ballot(valid && !(smallest > keep)) == 0) continue;        // wave-uniform
                uint32_t open = 0;
#pragma unroll
                for (int q = 0; q < 16; ++q) open |= (uint32_t)(!(__builtin_fabsf(z[q]) > keep)) << q;
                if (!valid) open = 0;
                if (any_zeros && keep < __builtin_inff()) open &= ~(uint32_t)reinterpret_cast<const uint16_t *>(zero_columns)[bit0 / 16];
                // rows with open bits go out for the chain: both lanes of such a row have half of it
                const uint64_t any = __ballot(open != 0);
                if ((any >> fr | any >> (fr + 32)) & 1u) {
                    int of_lane = lane;
                    asm volatile("" : "+v"(of_lane));        // (the address is made here, not kept: the registers are needed)
                    float *to = rows + (size_t)(m + 32 * i + (of_lane & 31)) * part_width + of_pair * 32 + 4 * (of_lane >> 5);
#pragma unroll
                    for (int q = 0; q < D / 8; ++q)
                        *reinterpret_cast<v4f *>(to + 8 * q) = v4f{value(q >> 2, 4 * (q & 3)), value(q >> 2, 4 * (q & 3) + 1),
                                                                   value(q >> 2, 4 * (q & 3) + 2), value(q >> 2, 4 * (q & 3) + 3)};
                }
                while (__ballot(open != 0) != 0) {           // wave-uniform
                    if (cnt + 64 > kList) work_off(std::integral_constant<int, 16>{});
                    const uint64_t pm = __ballot(open != 0);
                    if (open) {
                        const int pos = __builtin_ctz(open);
                        const int at = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(pm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pm, 0u));
                        list[at] = open_bit((uint32_t)row * (uint32_t)map.H + head, bit0 + pos, (bits >> pos) & 1u, second);
                        open &= open - 1u;
                    }
                    cnt += __builtin_popcountll(pm);
                }
            }
        });
        work_off(std::integral_constant<int, D>{});
    }
};

template <int D, int NB>
int launch(const GemmArgs &g, const Epilogue &e, const float *proj, const Tensors &of, const RowMap &map, bool wide, hipStream_t st) {
    const HashStore<D, NB> store(e, proj, of, map);
    if (wide) return launch_tile<NtTile<I8Traits, 256, 128, 64, 2, 1>, 2>(g, store, st, "QKV projection and hash");
    return launch_tile<NtTile<I8Traits, 128, 128, 64, 2, 1>, NB == 256 ? 2 : 3>(g, store, st, "QKV projection and hash");
}

}  // namespace

// Whole layers with the projection and the hash as launches of their own (with the LayerNorm in the projection where norm_linear.hip
// takes it) and with this one, linear attention, MLP of E (E <= 256: 4E), us:
//   E = 384   64 bits: 197 rows 37.9, 37.0; 1379 49.8, 46.6; 6304 84.3, 77.8; 12608 109.5, 100.8; 40000 258.0, 220.0
//            128 bits: 394 rows 46.2, 46.6; 1379 57.4, 53.7; 12608 121.5, 110.0.  256 bits: 788 rows 55.4, 56.4; 12608 138.7, 130.7
//   E = 768   64 bits: 197 rows 39.8, 40.2; 394 48.5, 46.8; 12608 216.8, 201.0; 25216 419.6, 366.2
//            128 bits: 591 rows 54.9, 55.5; 1379 71.7, 70.3; 12608 232.5, 222.4.  256 bits: 1379 rows 77.9, 77.4; 12608 264.8, 262.8
//   E = 256   64 bits: 3152 rows 57.9, 52.4; 10047 87.3, 79.1; 18000 106.8, 96.7; 25216 116.8, 116.9; 32768 128.9, 130.8; 50176 227.1, 201.4
//            256 bits: 1970 rows 57.7, 58.9; 3152 66.8, 65.2; 20000 134.9, 135.1; 32768 169.7, 182.0; 50176 275.9, 269.0
//   E = 192   64 bits: 4500 rows 57.7, 51.5; 20000 86.8, 81.5; 32768 105.3, 111.3; 65536 191.3, 177.2
//            256 bits: 3152 rows 64.5, 63.4; 20000 111.5, 109.7; 25216 119.7, 123.3; 65536 258.3, 263.9
//   E = 128  128 bits: 18000 rows 65.2, 60.7; 65536 130.6, 133.6; 90000 169.9, 166.2.  256 bits: 4096 rows 47.2, 50.2; 65536 151.5, 165.1
// From a few hundred rows on, as the hash's share of a tile is the same for few rows; not between 20480 rows and where Q, K and V outgrow
// the cache behind L2 (until then their way through memory costs less than what the tiles wait for each other) for narrow rows.
// Packed weights are decoded first, in a launch with those of the MLP, which as three launches rode in the hash's: from more rows on.
//   E = 768   64 bits: 3152 rows 93.8, 93.7; 6304 130.3, 123.0; 12608 217.7, 195.2.  128 bits: 3152 98.4, 99.3; 12608 238.7, 221.4
//            256 bits: 3152 rows 118.3, 118.0; 12608 270.9, 259.1
//   E = 384  128 bits: 1576 rows 58.3, 60.0; 12608 115.4, 110.2; 50176 344.4, 310.9
//   E = 256  128 bits: 6304 rows 71.2, 73.1; 12608 86.1, 82.6; 131072 528.0, 485.5.  256 bits: 12608 99.8, 99.0; 131072 607.9, 579.8
//   E = 192   64 bits: 3152 rows 53.2, 53.8; 12608 68.7, 64.7; 131072 387.1, 353.1.  256 bits: 50176 217.9, 218.4
//   E =  64   64 bits: 12608 rows 37.8, 38.0; 131072 118.1, 111.1.  256 bits: 131072 153.2, 164.6
//
// A tile with the hash behind its sums takes long, and the more bits the longer, so a last round of few tiles costs more than its launch
// saves.  From 4000 layers with linear attention, both ways on the same buffers, separate launches / one:
//   128 bits or heads of 32: 1024 x 322 rows 55.1 / 58.6 (64 bits 1024 x 420 67.0 / 68.6), 1024 x 669 69 / 67.5; 640 x 505 56.8 / 59.3
//   256 bits, prepared: rows in tiles of 128 that are one for half of the CUs, 384 x 1330 63.8 / 66.6, 512 x 1784 71 / 72.5, two for most, 512 x
//     5122 122 / 117, 1024 x 2739 159 / 150, or three, 640 x 4826 140 / 144, 896 x 4200 1.023, 448 x 8474 1.030; at 192 columns a second tile
//     for few CUs, 6501 1.013, 7289 1.015 (256 x 5586 88.0 / 84.7)
//   256 bits, packed: up to 1.7 rounds of the taller tiles 384 x 20169 206 / 213, 768 x 10565 287 / 296, 1024 x 5805 216 / 227; 256 columns up
//     to 85000 rows 35351 208 / 213, 66248 381 / 394, but 90138 455 / 430
//   widths of 320, 640 and 1280 gain least, and lose where a second round begins: 320 x 12069, 256 bits, packed 134 / 141, 16665 165 / 181, prepared
//     18060 1.035; 128 bits packed 320 x 17838 148 / 152, 640 x 8251 180 / 183; 64 bits 320 x 17038 132 / 135; elsewhere 640 x 17875, 128 bits, 0.92
//   packed 64 columns: 128 bits 72420 rows 125 / 131, 116472 144 / 146; two heads 70228 82 / 84; 64 bits 67792 1.025, 81952 1.010, 99356 0.969
bool sa::linear_hash_one_launch(long T, int E, int H, int nbits, bool packed) {
    const int d = E / H;
    if (!((d == 32 && nbits == 64) || (d == 64 && (nbits == 64 || nbits == 128 || nbits == 256))) || E % 64 != 0 || T * H >= (1L << 31)) return false;
    const long cols = (3L * E + 127) / 128, tiles = (T + 127) / 128 * cols, tall = (T + 255) / 256 * cols;     // (see launch_linear_hash)
    const bool least = E % 320 == 0;
    if (packed) {
        if (nbits == 256) return E >= 384 ? tall >= 870 && E <= 1024 : E == 256 && T * E >= 22L << 20;
        if (T * E < 3L << 20) return false;
        if (E == 64) return d == 64 && nbits == 64 && (tall <= 512 || tall >= 700);
        return !least || tall <= 480 || tall >= (nbits == 64 ? 700 : 780);
    }
    if (E <= 256) {
        if (T > 20480 && (T * E < 10L << 20 || (nbits == 256 && E < 256))) return false;
        if (nbits == 256) return T * E >= 650L << 10 && (E == 256 || tiles < 255 || tiles >= 330);
    } else if (nbits == 256) {
        if (T < 1900 || E > 1024) return false;
        if (tiles <= 768) return tiles <= (least ? 490 : 660);
        return !least || tall <= 512 || (E > 320 && tall >= 780);
    }
    if (nbits == 64 && d == 64 && E <= 640) return T >= 300;
    return T >= 640 && (E <= 512 || tiles >= 110);
}

int sa::launch_linear_hash(const int8_t *codes, int B, int N, int H, int E, const int8_t *wqkv_planes, float scale, const float *proj, int nbits,
                           float *q, float *k, uint64_t *q_codes, uint64_t *k_codes, float *v, hipStream_t st) {
    GemmArgs g;
    g.a = codes;
    g.gather_a = false;
    g.b[0] = wqkv_planes;
    g.b[1] = wqkv_planes + (size_t)3 * E * E;
    g.sel = RowSel{nullptr, nullptr, 0, (long)B * N};
    g.K = E;
    g.N = 3 * E;
    Epilogue e;
    e.parts[0] = e.parts[1] = e.parts[2] = v;                // only column block 2 is written whole
    e.part_width = E;
    e.lin_scale = scale;
    const Tensors of{q, k, q_codes, k_codes};
    const RowMap map{FastDiv((uint32_t)H), FastDiv((uint32_t)N), N, H, nbits / 64};
    // 128 x 128 up to a round of them, three per CU, then 256 x 128 (64 and 128 bits, us: 5122 x 384 67.4, 70.4 and 74.1, 77.1; 12608 x 384
    // 99.8, 100.8 and 114.0, 110.0; 6304 x 768 130.2, 124.6 and 143.3, 140.4; 20000 x 768 273.5, 269.1 and 313.0, 307.5)
    const bool wide = (g.sel.max_rows + 127) / 128 * ((g.N + 127) / 128) > 768;
    if (E == 32 * H) return launch<32, 64>(g, e, proj, of, map, wide, st);
    switch (nbits) {
        case 64: return launch<64, 64>(g, e, proj, of, map, wide, st);
        case 128: return launch<64, 128>(g, e, proj, of, map, wide, st);
    }
    return launch<64, 256>(g, e, proj, of, map, wide, st);
}
