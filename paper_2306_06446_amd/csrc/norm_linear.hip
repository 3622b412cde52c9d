// LayerNorm and the Q, K, V projection of a layer in one launch, for widths whose rows a workgroup can hold (E = 64 .. 256):
//     (q, k, v)[row] = scale * Wqkv . codes(LayerNorm(x[row]))
// Every wavefront normalises its share of a workgroup's 64 rows into codes in LDS, from where all of them take theirs as operands;
// the planes of Wqkv stream past, 64 to 128 rows of one plane at a time, and a plane pair's sums leave from the registers.
//
// Bound by the outputs, 12 bytes per element of x, and for few rows by the weights, all of which a workgroup passes through its
// CU.  Two workgroups share a CU, so that one multiplies while the other writes (units of E rows and one workgroup per CU: layer
// of 65536 rows x 192 214 us, 196 with two).  As a launch each the LayerNorm wrote codes that every column tile of the projection
// read again.  Layer, two launches -> one:
//   25088 x  64 (32 images)  42.3 -> 39.0 us     65536 x  64   70.9 -> 62.6
//   25088 x 128              68.6 -> 64.8        65536 x 128  126.6 -> 112.0
//   25088 x 192             109.0 -> 98.9        65536 x 192  204.0 -> 194.1
//   16384 x 256             113.8 -> 106.3       65536 x 256  257.4 -> 250.5
#include "common.h"
#include "gemm_common.h"
#include "gemm_mfma.h"
#include "layernorm.h"

namespace {

using namespace sa;

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8, kMI = 2, kRows = 32 * kMI;        // wavefronts 2 x 4 over rows x columns, 16-row tiles of each, rows

// NE: E / 64.  TN: 16-column tiles of a wavefront in a unit.
template <int NE>
struct NormLinearShape {
    static constexpr int E = 64 * NE, TN = NE == 3 ? 1 : NE == 4 ? 2 : NE, ROWS = 64 * TN, UNIT = ROWS * E;       // rows of one plane
    static constexpr int UNITS = 6 * E / ROWS, RING = NE == 1 ? 6 : NE == 2 ? 3 : NE == 3 ? 4 : 2;
    static constexpr int TOTAL = UNIT / 1024, LOADS = (TOTAL + kWaves - 1) / kWaves;       // KiB of a unit, of a wavefront
    static constexpr int CODES = RING * UNIT, LDS_BYTES = CODES + kRows * E;
    static_assert(2 * LDS_BYTES <= 160 * 1024, "two workgroups to a CU");
};

template <int NE>
__global__ __launch_bounds__(kWaves * 64) void norm_linear_kernel(NormRows norm, long n_rows, const int8_t *__restrict__ w, float scale,
                                                                  float *__restrict__ q, float *__restrict__ k, float *__restrict__ v) {
    using S = NormLinearShape<NE>;
    constexpr int E = S::E;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[S::LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 2, wc = wave & 3, fr = lane & 15, fg = lane >> 4;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    const long m0 = (long)blockIdx.x * kRows;
    if (blockIdx.x == 0) zero_words(norm.zero);

    // this wavefront's rows, LPR lanes each
    constexpr int LPR = NE == 1 ? 16 : NE == 2 ? 32 : 64, GROUPS = 64 / LPR, STEPS = kRows / kWaves / GROUPS;
    const int l = lane % LPR, row0 = wave * (kRows / kWaves) + lane / LPR;
    const bool in = 4 * l < E;
    const int col = min(4 * l, E - 4);                                   // (lanes past the row: its end, not used; see row_or_zero)
    float4 xr[STEPS];
#pragma unroll
    for (int i = 0; i < STEPS; ++i)
        xr[i] = *reinterpret_cast<const float4 *>(norm.x + (size_t)min(m0 + row0 + GROUPS * i, n_rows - 1) * E + col);
    const float4 gamma = *reinterpret_cast<const float4 *>(norm.gamma + col);
    const float4 beta = *reinterpret_cast<const float4 *>(norm.beta + col);

    // unit u: plane u % 2 of columns u / 2 ROWS ..
    auto issue = [&](int u, int slot) {
        const int8_t *base = w + (size_t)(u % 2) * 3 * E * E + (size_t)(u / 2) * S::UNIT;
#pragma unroll
        for (int j = 0; j < S::LOADS; ++j) {
            const int kib = (j * kWaves + wave) % S::TOTAL;              // (past the end: the same bytes once more)
            const int c = kib * 64 + lane, r = c / (4 * NE);
            direct_load_16(base, (uint32_t)(r * E + swizzle_row<NE>(r, c % (4 * NE)) * 16), lds_base + slot * S::UNIT + kib * 1024);
        }
    };
#pragma unroll
    for (int u = 0; u < S::RING; ++u) issue(u, u);

#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        const float4 x[1] = {row_or_zero(xr[i], in)};
        float mean, rstd, y[4];
        row_stats<LPR, 1>(x, l, E, norm.eps, mean, rstd);
        normalise(x[0], mean, rstd, gamma, beta, y);
        const int r = row0 + GROUPS * i;
        if (in) *reinterpret_cast<uint32_t *>(lds + S::CODES + r * E + swizzle_row<NE>(r, l / 4) * 16 + l % 4 * 4) = codes_of(y, norm.inv_scale);
    }
    __syncthreads();
    uint4 xf[kMI][NE];
#pragma unroll
    for (int i = 0; i < kMI; ++i)
#pragma unroll
        for (int s = 0; s < NE; ++s) {
            const int r = wr * 16 * kMI + 16 * i + fr;
            xf[i][s] = *reinterpret_cast<const uint4 *>(lds + S::CODES + r * E + swizzle_row<NE>(r, 4 * s + fg) * 16);
        }

    // Products are computed transposed (weights down, rows across): a lane holds four consecutive columns of row lane % 16.
    v4i acc[kMI][S::TN];
    static_for<S::UNITS>([&](auto u_c) {
        constexpr int u = decltype(u_c)::value, slot = u % S::RING;
        constexpr int later = (S::UNITS < u + S::RING ? S::UNITS : u + S::RING) - 1 - u;       // units on their way behind this one
        if constexpr (u == 0 || S::RING < S::UNITS) {
            wait_loads_in_flight<S::RING < S::UNITS ? later * S::LOADS : 0>();
            __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < NE; ++s)
#pragma unroll
            for (int t = 0; t < S::TN; ++t) {
                const int r = wc * 16 * S::TN + 16 * t + fr;
                const uint4 b = *reinterpret_cast<const uint4 *>(lds + slot * S::UNIT + r * E + swizzle_row<NE>(r, 4 * s + fg) * 16);
#pragma unroll
                for (int i = 0; i < kMI; ++i)
                    acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, b), __builtin_bit_cast(v4i, xf[i][s]),
                                                                      u % 2 == 0 && s == 0 ? v4i{0, 0, 0, 0} : acc[i][t], 0, 0, 0);
            }
        if constexpr (u + S::RING < S::UNITS) {
            __syncthreads();                                             // this unit has been read
            issue(u + S::RING, slot);
        }
        if constexpr (u % 2 == 1) {
            constexpr int c0 = u / 2 * S::ROWS;
            float *out = (c0 < E ? q : c0 < 2 * E ? k : v) + c0 % E + wc * 16 * S::TN + 4 * fg;
#pragma unroll
            for (int i = 0; i < kMI; ++i) {
                const long m = m0 + wr * 16 * kMI + 16 * i + fr;
                if (m < n_rows) {
#pragma unroll
                    for (int t = 0; t < S::TN; ++t)
                        *reinterpret_cast<float4 *>(out + (size_t)m * E + 16 * t) =
                            make_float4(__builtin_fmaf((float)acc[i][t][0], scale, 0.0f), __builtin_fmaf((float)acc[i][t][1], scale, 0.0f),
                                        __builtin_fmaf((float)acc[i][t][2], scale, 0.0f), __builtin_fmaf((float)acc[i][t][3], scale, 0.0f));
                }
            }
        }
    });
}

template <int NE>
int launch(const NormRows &norm, long T, const int8_t *w, float scale, float *q, float *k, float *v, hipStream_t st) {
    const long blocks = (T + kRows - 1) / kRows;
    SA_REQUIRE(blocks < (1L << 31), SA_ERR_SHAPE, "layer: too many rows for one launch");
    norm_linear_kernel<NE><<<dim3((unsigned)blocks), dim3(kWaves * 64), 0, st>>>(norm, T, w, scale, q, k, v);
    return check_launch("LayerNorm and QKV projection");
}

}  // namespace

// Whether one launch is the faster way: with few rows, and so few workgroups, the weights take longer through each of them than
// two launches.  Layers of 192, two launches against one: 197 rows 34.5 and 40.2 us, 9456 rows 56.9 and 59.2, 10000 rows 57.3 and
// 59.0, 10500 rows 60.4 and 59.6, 12288 rows 64.5 and 63.0; of 256: 10240 rows 69.1 both, 12608 rows 72.9 and 72.3, 16384 rows
// 80.5 and 75.6; 788 x 128 35.9 and 36.5, 1576 x 128 38.0 and 37.8.  At E = 64 they are 24 KiB (197 rows: 24.9 and 22.8).  (Where
// a few CUs have one workgroup more than the others it is slower by up to 3 % all the same: 17000 x 192 81.6 and 83.9, 20000 x 192
// 87.0 and 85.2.)
bool sa::norm_linear_one_launch(long T, int E) {
    if (E > 256 || E % 64 != 0) return false;
    return E == 64 || T >= (E == 128 ? 12L : 54L) * E;
}

int sa::launch_norm_linear(const NormRows &norm, long T, int E, const int8_t *wqkv_planes, float scale, float *q, float *k, float *v,
                           hipStream_t st) {
    // (In the order they lie in the code object.  The widest, whose unrolled loop is 12 KB of instructions, takes 5 % longer where it
    // starts at an even multiple of 256 bytes: layer of 65536 x 256 249 us first, 256 last.)
    switch (E) {
        case 256: return launch<4>(norm, T, wqkv_planes, scale, q, k, v, st);
        case 64: return launch<1>(norm, T, wqkv_planes, scale, q, k, v, st);
        case 128: return launch<2>(norm, T, wqkv_planes, scale, q, k, v, st);
        case 192: return launch<3>(norm, T, wqkv_planes, scale, q, k, v, st);
    }
    return fail(SA_ERR_UNSUPPORTED, "layer: width %d with the LayerNorm in the projection", E);
}
