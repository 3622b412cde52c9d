// Both experts of a two-expert MoE layer by layer (Sec. 4.2): one launch holds the tiles of the Shift expert (int8 x two
// weight planes) and those of the Mult expert (fp16) for the tokens each was given.
#include "common.h"
#include "gemm_common.h"
#include "gemm_mfma.h"
#include "gemm_stores.h"

namespace {

using namespace sa;

constexpr int kPlaces = 64;                                  // of an XCD: two workgroups on each of its 32 CUs

// Tiles of an XCD: `cols` of every row of tiles, of which it has one of 1 << log_rg.
struct XcdTiles {
    int cols, log_rg;
    __device__ explicit XcdTiles(const GemmArgs &g) : cols(g.cols_per_group), log_rg(3 - g.log_groups) {}
    // rows of tiles of the fullest XCD, tiles of all XCDs
    template <class Tile>
    __device__ int rows(long n) const {
        return (int)((((uint32_t)n + Tile::BM - 1) / Tile::BM + (1u << log_rg) - 1) >> log_rg);
    }
    template <class Tile>
    __device__ int blocks(long n) const { return 8 * rows<Tile>(n) * cols; }
};

// How many of the Shift expert's rows go to its higher tiles.  A CU's two workgroups share its matrix cores, so a CU with two of the higher tiles is
// done last.  If all tiles are one round of workgroups and some CUs would have two of the higher ones: only as many of these as there are CUs.
template <class TileS, class TileL, class TileM>
__device__ inline long split_shift_rows(long n_shift, const XcdTiles &s, long n_mult, const XcdTiles &m, int most) {
    const int tiles_s = s.rows<TileS>(n_shift) * s.cols, tiles_m = m.rows<TileM>(n_mult) * m.cols;
    const long high = (long)(most << s.log_rg) * TileS::BM;              // most: rows of tiles that 32 CUs have
    if (tiles_s <= kPlaces / 2 || tiles_s + tiles_m > kPlaces || high <= 0 || high >= n_shift) return n_shift;
    return most * s.cols + s.rows<TileL>(n_shift - high) * s.cols + tiles_m <= kPlaces ? high : n_shift;
}

// How many of the Mult expert's rows go to its higher tiles: those of whole rounds of workgroups, if lower tiles take the other rows in one more.
template <class TileS, class TileM, class TileL>
__device__ inline long split_mult_rows(long n_shift, const XcdTiles &s, long n_mult, const XcdTiles &m) {
    const int tiles_s = s.rows<TileS>(n_shift) * s.cols, rows_m = m.rows<TileM>(n_mult), all = tiles_s + rows_m * m.cols, over = all % kPlaces;
    if (over == 0 || all < kPlaces) return n_mult;
    int left = rows_m;                                       // rows of higher tiles
    for (int t = over; t > 0; t -= m.cols) --left;
    const long high = (long)(left << m.log_rg) * TileM::BM;
    if (left <= 0) return n_mult;
    const int places = kPlaces + all - over - (tiles_s + left * m.cols);
    return m.rows<TileL>(n_mult - high) * m.cols <= places ? high : n_mult;
}

// Workgroups of the Shift expert first, the Mult expert's behind them.  How many tiles either has is known on the device
// only (the routing counts): a workgroup past the end of both leaves.
template <class TileS, class StoreS, class TileM, class StoreM, int OCC>
__global__ __launch_bounds__(256, OCC) void expert_pair_kernel(GemmArgs gs, StoreS ss, GemmArgs gm, StoreM sm) {
    constexpr int LDS_S = TileS::template lds_bytes<StoreS>(), LDS_M = TileM::template lds_bytes<StoreM>();
    constexpr int LDS_BYTES = LDS_S > LDS_M ? LDS_S : LDS_M;
    static_assert(LDS_BYTES * OCC <= 160 * 1024, "OCC workgroups of these tiles do not fit the LDS of a CU");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_BYTES];
    const int32_t *rows;
    long n_shift;
    resolve_rows(gs.sel, rows, n_shift);
    const int shift_blocks = XcdTiles(gs).blocks<TileS>(n_shift);      // a multiple of 8
    if ((int)blockIdx.x < shift_blocks)
        TileS::template run<StoreS>(gs, ss, blockIdx.x, lds);
    else
        TileM::template run<StoreM>(gm, sm, (int)blockIdx.x - shift_blocks, lds);
}

// The same with two heights of one expert's tiles: its last rows go to the lower ones, where that fills the last round of workgroups better.
// 12608 tokens, 70 % of them to the Shift expert: 3072 <- 768 has 840 + 480 tiles for 512 places, and 48 CUs with a sixth tile took 18 us longer
// than the others (73 us by the tiles' own clocks; with 80 % of the Mult rows in lower tiles 67); 768 <- 3072 has 315 + 180, and the CUs with two high
// Shift tiles were done 8 us after the others (61 and 58).  Of that the clock takes half back, the card being at its power limit: block 201.4 ->
// 197.4 us (50 %: 224.6, 224.1), layer 315.7 -> 308.6; block of 18912 tokens, 50 %, 302.9 -> 300.6; where no rows are taken the same as without (4728
// to 15760 tokens within 0.5 %).
// SPLIT_SHIFT: the Shift expert's (TileL: its lower tiles), else the Mult expert's.
template <class TileS, class StoreS, class TileM, class StoreM, class TileL, bool SPLIT_SHIFT, int OCC>
__global__ __launch_bounds__(256, OCC) void expert_split_kernel(GemmArgs gs, StoreS ss, GemmArgs gm, StoreM sm, int most) {
    typedef typename std::conditional<SPLIT_SHIFT, StoreS, StoreM>::type StoreL;
    constexpr int LDS_S = TileS::template lds_bytes<StoreS>(), LDS_M = TileM::template lds_bytes<StoreM>(), LDS_L = TileL::template lds_bytes<StoreL>();
    constexpr int LDS_SM = LDS_S > LDS_M ? LDS_S : LDS_M, LDS_BYTES = LDS_SM > LDS_L ? LDS_SM : LDS_L;
    static_assert(LDS_BYTES * OCC <= 160 * 1024, "OCC workgroups of these tiles do not fit the LDS of a CU");
    static_assert(TileL::BN == TileS::BN && TileL::BN == TileM::BN, "one walk over the columns");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_BYTES];
    const int32_t *rows;
    long n_shift, n_mult;
    resolve_rows(gs.sel, rows, n_shift);
    resolve_rows(gm.sel, rows, n_mult);
    const XcdTiles xs(gs), xm(gm);
    const long high = SPLIT_SHIFT ? split_shift_rows<TileS, TileL, TileM>(n_shift, xs, n_mult, xm, most)
                                  : split_mult_rows<TileS, TileM, TileL>(n_shift, xs, n_mult, xm);
    const int s_blocks = xs.blocks<TileS>(SPLIT_SHIFT ? high : n_shift), m_blocks = xm.blocks<TileM>(SPLIT_SHIFT ? n_mult : high);
    int b = blockIdx.x;                                      // (all of them multiples of 8)
    if (b < s_blocks) return TileS::template run<StoreS>(gs, ss, b, lds, 0, SPLIT_SHIFT ? high : n_shift);
    b -= s_blocks;
    if constexpr (SPLIT_SHIFT) {
        const int l_blocks = xs.blocks<TileL>(n_shift - high);
        if (b < l_blocks) return TileL::template run<StoreS>(gs, ss, b, lds, high);
        TileM::template run<StoreM>(gm, sm, b - l_blocks, lds);
    } else {
        if (b < m_blocks) return TileM::template run<StoreM>(gm, sm, b, lds, 0, high);
        TileL::template run<StoreM>(gm, sm, b - m_blocks, lds, high);
    }
}

// Both experts' tiles one round of workgroups: the Shift expert's last rows in tiles of half the height (even_rows).
template <class TileS, class StoreS, class TileM, class StoreM, class TileL, int OCC>
__global__ __launch_bounds__(256, OCC) void expert_even_kernel(GemmArgs gs, StoreS ss, GemmArgs gm, StoreM sm) {
    constexpr int LDS_S = TileS::template lds_bytes<StoreS>(), LDS_M = TileM::template lds_bytes<StoreM>(), LDS_L = TileL::template lds_bytes<StoreS>();
    constexpr int LDS_SM = LDS_S > LDS_M ? LDS_S : LDS_M, LDS_BYTES = LDS_SM > LDS_L ? LDS_SM : LDS_L;
    static_assert(LDS_BYTES * OCC <= 160 * 1024, "OCC workgroups of these tiles do not fit the LDS of a CU");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_BYTES];
    const int32_t *rows;
    long n_shift, n_mult;
    resolve_rows(gs.sel, rows, n_shift);
    resolve_rows(gm.sel, rows, n_mult);
    const XcdTiles xs(gs), xm(gm);
    const int m_tiles = xm.rows<TileM>(n_mult) * xm.cols, m_blocks = 8 * m_tiles;
    const long high = even_rows<TileS::BM, OCC>((uint32_t)n_shift, gs, m_tiles);
    int b = blockIdx.x;                                      // (all of them multiples of 8)
    const int s_blocks = xs.blocks<TileS>(high);
    if (b < s_blocks) return TileS::template run<StoreS>(gs, ss, b, lds, 0, high);
    b -= s_blocks;
    if (b < m_blocks) return TileM::template run<StoreM>(gm, sm, b, lds);
    TileL::template run<StoreS>(gs, ss, b - m_blocks, lds, high);
}

template <class TileS, class TileM, int OCC, class StoreS, class StoreM>
int launch_pair_tiles(const GemmArgs &gs, const StoreS &ss, const GemmArgs &gm, const StoreM &sm, hipStream_t st, const char *what) {
    GemmArgs s = gs, m = gm;
    s.share_out(TileS::BN, TileS::col_groups(gs));
    m.share_out(TileM::BN, TileM::col_groups(gm));
    // the rows of both add up to max_rows: all on either side, and one more row of tiles per XCD where the other side starts
    const long all_s = tile_blocks<TileS>(gs.sel.max_rows, s), all_m = tile_blocks<TileM>(gm.sel.max_rows, m);
    const long step_s = tile_blocks<TileS>(1, s), step_m = tile_blocks<TileM>(1, m);
    const long blocks = (all_s > all_m ? all_s : all_m) + step_s + step_m;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "%s: too many tiles for one launch", what);
    expert_pair_kernel<TileS, StoreS, TileM, StoreM, OCC><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(s, ss, m, sm);
    return check_launch(what);
}

template <class TileS, class TileM, class TileL, int OCC, class StoreS, class StoreM>
int launch_even_tiles(const GemmArgs &gs, const StoreS &ss, const GemmArgs &gm, const StoreM &sm, hipStream_t st, const char *what) {
    GemmArgs s = gs, m = gm;
    s.share_out(TileS::BN, TileS::col_groups(gs));
    m.share_out(TileM::BN, TileM::col_groups(gm));
    if (!may_be_even<TileS::BM, TileM::BM, OCC>(s, m, gs.sel.max_rows)) return launch_pair_tiles<TileS, TileM, OCC>(gs, ss, gm, sm, st, what);
    // as launch_pair_tiles, and the lower tiles: at most one a CU and two for each of a row of tiles (even_rows)
    const long all_s = tile_blocks<TileS>(gs.sel.max_rows, s), all_m = tile_blocks<TileM>(gm.sel.max_rows, m);
    const long step_s = tile_blocks<TileS>(1, s), step_m = tile_blocks<TileM>(1, m);
    const long blocks = (all_s > all_m ? all_s : all_m) + 3 * step_s + step_m + 256;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "%s: too many tiles for one launch", what);
    expert_even_kernel<TileS, StoreS, TileM, StoreM, TileL, OCC><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(s, ss, m, sm);
    return check_launch(what);
}

template <class TileS, class TileM, class TileL, bool SPLIT_SHIFT, int OCC, class StoreS, class StoreM>
int launch_split_tiles(const GemmArgs &gs, const StoreS &ss, const GemmArgs &gm, const StoreM &sm, hipStream_t st, const char *what) {
    GemmArgs s = gs, m = gm;
    s.share_out(TileS::BN, TileS::col_groups(gs));
    m.share_out(TileM::BN, TileM::col_groups(gm));
    // Shift rows are taken of one round of workgroups.  Mult rows of any last round, but behind five others that is no more than workgroups lose
    // by asking (768 -> 3072, 30 / 50 / 70 %, us without and with: 30000 tokens 173.4 / 172.5 / 166.1, 174.8 / 172.3 / 166.1; 40000 227.6 /
    // 224.0 / 218.8, 229.9 / 225.8 / 217.7; 60000 335.3 / 330.8 / 311.5, 340.1 / 327.9 / 313.1; 25000 147.7 / 149.0 / 143.7, 148.9 / 147.4 / 142.1).
    if (least_tiles<TileS::BM, TileM::BM>(s, m, gs.sel.max_rows) > (SPLIT_SHIFT ? 1 : 5) * kPlaces)
        return launch_pair_tiles<TileS, TileM, OCC>(gs, ss, gm, sm, st, what);
    // as launch_pair_tiles, and what the lower tiles take: at most a round of workgroups more, and a row of tiles per XCD
    const long all_s = tile_blocks<TileS>(gs.sel.max_rows, s), all_m = tile_blocks<TileM>(gm.sel.max_rows, m);
    const long step_s = tile_blocks<TileS>(1, s), step_m = tile_blocks<TileM>(1, m);
    const long blocks = (all_s > all_m ? all_s : all_m) + 2 * (step_s + step_m) + 8 * kPlaces;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "%s: too many tiles for one launch", what);
    expert_split_kernel<TileS, StoreS, TileM, StoreM, TileL, SPLIT_SHIFT, OCC>
        <<<dim3((unsigned)blocks), dim3(256), 0, st>>>(s, ss, m, sm, kPlaces / 2 / s.cols_per_group);
    return check_launch(what);
}

// Tile choice.  Up to 640 tiles of 64 x 64 the small tiles of gemm_slice.h, by the lines launch_gemm draws for the rows of
// both experts together; beyond, from a sweep over routings of 30 / 50 / 70 % (12608 tokens unless said, one launch for both
// experts against one each):
//    768 -> 3072  256 x 128 and 192 x 128   112 / 109 / 105 us (128 x 128: 126 / 123 / 116; apart 131 / 130 / 112)
//   3072 ->  768  192 x 128 both             82 /  81 /  77 us (128 x 128:  97 /  94 /  86; apart 121 / 120 /  88).  Of the Mult
//                 tiles 120 then shared a CU with a Shift tile each and were done 20 us after it: as 128 x 128, with a ring of four
//                 short stages, the whole block 215 -> 210 us, the layer 345 -> 338
//    768 ->  768  128 x 128 both             34 /  35 /  33 us (192 x 128:  34 /  34 /  34; apart  49 /  47 /  49)
//    384 -> 1536                128 x 128 both  44 / 41 / 42 us    (192 x 128:  46 /  46 /  47; apart  64 /  66 /  55)
//   1536 ->  384, 384 -> 384    128 x 64 and 64 x 128   33 and 16 us   (128 x 128: 35 and 20; apart 48 and 35)
//   131072 tokens 256 -> 1024               238 us             (256 x 128: 251; apart 275)
// Few tokens with whole-line stages take 32 x 32 tiles, as in launch_gemm (block of 197 tokens x 192, 768 hidden 24.0 -> 23.6 us,
// 197 x 768, 3072 hidden 31.9 -> 31.1, 1 x 768 23.3 -> 20.7; 300 x 768, fifteen tiles for sixteen CUs: 38.4 both).
enum class PairTiles { kSlice32x32, kSlice32, kSlice64, kLarge, kLongRows, kFine, kMiddle };

// rows of whole 128-byte lines, at least four of them
bool shift_lines(const GemmArgs &gs) { return gs.K % 128 == 0 && (gs.a_valid == 0 || gs.a_valid == gs.K) && gs.K >= 512; }
bool mult_lines(const GemmArgs &gm) { return gm.K % 64 == 0 && gm.K >= 256; }

PairTiles choose_pair(const GemmArgs &gs, const GemmArgs &gm) {
    const bool lines_s = shift_lines(gs), lines_m = mult_lines(gm);
    auto tiles = [&](long bm, long bn) { return ((gs.sel.max_rows + bm - 1) / bm) * ((gs.N + bn - 1) / bn); };
    if (lines_s && tiles(32, 32) <= 192) return PairTiles::kSlice32x32;
    if (tiles(32, 64) <= 256) return PairTiles::kSlice32;
    if (tiles(64, 64) <= 640) return PairTiles::kSlice64;
    // more than two rounds of the large Shift tile at two per CU: its higher rate counts for more than an even last round
    if (lines_s && lines_m && tiles(256, 128) > 1024) return PairTiles::kLarge;
    if (lines_s && lines_m && gs.K >= 2048) return PairTiles::kLongRows;
    // not half of the chip's 768 places: finer tiles
    if (lines_m && tiles(128, 128) <= 384) return PairTiles::kFine;
    return PairTiles::kMiddle;
}

template <class StoreS, class StoreM>
int launch_pair(const GemmArgs &gs, const StoreS &ss, const GemmArgs &gm, const StoreM &sm, hipStream_t st, const char *what) {
    typedef I8Traits I;
    typedef F16Traits F;
    const bool lines_s = shift_lines(gs), lines_m = mult_lines(gm);
    switch (choose_pair(gs, gm)) {
        case PairTiles::kSlice32x32:
            return launch_pair_tiles<SliceTile<I, 1, 1, 128, 5>, SliceTile<F, 1, 1, 128, 8>, 1>(gs, ss, gm, sm, st, what);
        case PairTiles::kSlice32:
            if (lines_s) return launch_pair_tiles<SliceTile<I, 1, 2, 128, 4>, SliceTile<F, 1, 2, 128, 6>, 1>(gs, ss, gm, sm, st, what);
            if (lines_m) return launch_pair_tiles<SliceTile<I, 1, 2, 64, 7>, SliceTile<F, 1, 2, 128, 6>, 1>(gs, ss, gm, sm, st, what);
            return launch_pair_tiles<SliceTile<I, 1, 2, 64, 7>, SliceTile<F, 1, 2, 64, 8>, 1>(gs, ss, gm, sm, st, what);
        case PairTiles::kSlice64:
            if (lines_s) return launch_pair_tiles<SliceTile<I, 2, 2, 128, 3>, SliceTile<F, 2, 2, 128, 4>, 2>(gs, ss, gm, sm, st, what);
            if (lines_m) return launch_pair_tiles<SliceTile<I, 2, 2, 64, 6>, SliceTile<F, 2, 2, 128, 4>, 2>(gs, ss, gm, sm, st, what);
            return launch_pair_tiles<SliceTile<I, 2, 2, 64, 6>, SliceTile<F, 2, 2, 64, 9>, 2>(gs, ss, gm, sm, st, what);
        case PairTiles::kLarge:
            return launch_split_tiles<NtTile<I, 256, 128, 64, 2, 1>, NtTile<F, 192, 128, 128, 2, 2>, NtTile<F, 128, 128, 128, 2, 2>, false, 2>(gs, ss, gm, sm, st, what);
        case PairTiles::kLongRows:
            if constexpr (StoreS::kScatter)                  // a second layer (the first one writes a hidden matrix)
                if (gs.a_block)
                    return launch_split_tiles<NtTile<I, 192, 128, 64, 2, 1, true>, NtTile<F, 128, 128, 64, 4, 1, true>, NtTile<I, 128, 128, 64, 3, 1, true>, true, 2>(
                        gs, ss, gm, sm, st, what);
            return launch_split_tiles<NtTile<I, 192, 128, 64, 2, 1>, NtTile<F, 128, 128, 64, 4, 1>, NtTile<I, 128, 128, 64, 3, 1>, true, 2>(gs, ss, gm, sm, st, what);
        case PairTiles::kFine:
            return launch_pair_tiles<NtTile<I, 128, 64, 64, 3, 1>, NtTile<F, 64, 128, 128, 2, 2>, 3>(gs, ss, gm, sm, st, what);
        case PairTiles::kMiddle: break;
    }
    return launch_even_tiles<NtTile<I, 128, 128, 64, 2, 1>, NtTile<F, 128, 128, 64, 3, 1>, NtTile<I, 64, 128, 64, 2, 1>, 3>(gs, ss, gm, sm, st, what);
}

GemmArgs args(const void *a, bool gather, const void *b0, const void *b1, const RowSel &sel, int K, int N) {
    GemmArgs g;
    g.a = a;
    g.gather_a = gather;
    g.b[0] = b0;
    g.b[1] = b1;
    g.sel = sel;
    g.K = K;
    g.N = N;
    return g;
}

}  // namespace

int sa::expert_pair_mlp(const ExpertPair &p, int E, int hid, const int8_t *w1_planes, const int8_t *w2_planes, const void *mw1,
                        const void *mw2, float requant_scale, const int8_t *lut, bool accumulate, int8_t *shift_hidden,
                        void *mult_hidden, hipStream_t st) {
    Epilogue s1, m1, s2, m2;
    s1.h = shift_hidden;
    s1.rq = requant_scale;
    s1.lut = lut;
    m1.hh = static_cast<_Float16 *>(mult_hidden);
    s2.yf = m2.yf = p.y;
    s2.gate = m2.gate = p.gate;
    s2.out_scale = p.out_scale;
    s2.accumulate = m2.accumulate = accumulate;
    GemmArgs gs2 = args(shift_hidden, false, w2_planes, w2_planes + (size_t)E * hid, p.shift_rows, hid, E);
    GemmArgs gm2 = args(mult_hidden, false, mw2, nullptr, p.mult_rows, hid, E);
    // The tiles for long rows take stages of 64 bytes of a row, half a line, which fill the LDS at half the rate of whole
    // lines.  Where the second layer has these tiles the hidden rows are laid out in columns of 64 bytes (a stage's rows are then
    // one behind the other): 12608 tokens, 768 <- 3072: 73 -> 68 us, the whole block 211.5 -> 207.7, the layer 344.1 -> 342.5.
    if (choose_pair(gs2, gm2) == PairTiles::kLongRows)
        s1.h_block = m1.h_block = gs2.a_block = gm2.a_block = (size_t)p.shift_rows.max_rows * 64;
    int rc = launch_pair(args(p.xq, true, w1_planes, w1_planes + (size_t)hid * E, p.shift_rows, E, hid), ShiftStore<kEpiRequantLut>(s1),
                         args(p.xh, true, mw1, nullptr, p.mult_rows, E, hid), MultStore<kEpiGeluHalf>(m1), st, "experts (fc1)");
    if (rc != SA_OK) return rc;
    return launch_pair(gs2, ShiftStore<kEpiScatterI32>(s2), gm2, MultStore<kEpiScatterF32>(m2), st, "experts (fc2)");
}

int sa::expert_pair_linear(const ExpertPair &p, int K, int N, const int8_t *w_planes, const void *w_f16, hipStream_t st) {
    Epilogue s, m;
    s.yf = m.yf = p.y;
    s.gate = m.gate = p.gate;
    s.out_scale = p.out_scale;
    const int Kp = (K + 63) / 64 * 64;                   // rows of the planes
    GemmArgs gs = args(p.xq, true, w_planes, w_planes + (size_t)N * Kp, p.shift_rows, Kp, N);
    gs.a_ld = gs.a_valid = K;
    return launch_pair(gs, ShiftStore<kEpiScatterI32>(s), args(p.xh, true, w_f16, nullptr, p.mult_rows, K, N),
                       MultStore<kEpiScatterF32>(m), st, "sa_moe_linear");
}
