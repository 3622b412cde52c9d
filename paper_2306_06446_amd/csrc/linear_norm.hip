// The output projection of a layer's attention and the second LayerNorm in one launch, for few rows of E = 64 .. 192 and prepared weights:
//     y[row] = residual[row] + scale * Wo . codes[row],     int8 codes, fp16 row and router logits of LayerNorm(y[row])
// A workgroup has 16 rows, a wavefront 16 of the columns.  Every load is asked for at its start and straight into registers (a wavefront is the
// only one of its workgroup to read its weights); the sums meet in LDS, where rows are taken as the kernel of layernorm.hip takes them: the
// same results.  Bound by its own chain: start, one round trip of loads, 2 to 6 products, a barrier, the sums of a row.  As two launches (4.3 +
// 3.4 us at 197 x 192) the second waits for the first to end, starts and reads y back: DeiT-Tiny layer of one image 39.0 -> 37.3 us.  With
// eight wavefronts at any width, some of two tiles, 37.7.
#include "common.h"
#include "gemm_common.h"
#include "layernorm.h"

namespace {

using namespace sa;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));

constexpr int kRows = 16;

template <int NE>
__global__ __launch_bounds__(NE * 256) void linear_norm_kernel(const int8_t *codes, NormRows norm, long n_rows, NormOut to) {
    constexpr int E = 64 * NE, WAVES = 4 * NE, PITCH = E + 4;            // a wavefront for 16 columns
    __shared__ __attribute__((aligned(16))) float rows_s[kRows * PITCH];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, fr = lane & 15, fg = lane >> 4;
    const long m0 = (long)blockIdx.x * kRows;
    const size_t m = (size_t)min(m0 + fr, n_rows - 1);

    // Products are computed transposed (weights down, rows across): a lane holds four consecutive columns of row lane % 16.
    uint4 a[NE], b[2][NE];
    const int col = 16 * wave + 4 * fg;
#pragma unroll
    for (int s = 0; s < NE; ++s) a[s] = *reinterpret_cast<const uint4 *>(codes + m * E + 64 * s + 16 * fg);
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int s = 0; s < NE; ++s) b[p][s] = *reinterpret_cast<const uint4 *>(norm.wo + (size_t)p * E * E + (16 * wave + fr) * E + 64 * s + 16 * fg);
    const float4 res = *reinterpret_cast<const float4 *>(norm.residual + m * E + col);
    // of the LayerNorm: LPR lanes a row
    constexpr int LPR = NE == 1 ? 16 : NE == 2 ? 32 : 64, LANES = 64 / LPR;
    const int l = lane % LPR, j = min(4 * l, E - 4);
    const bool in = 4 * l < E;
    const float4 gamma = *reinterpret_cast<const float4 *>(norm.gamma + j), beta = *reinterpret_cast<const float4 *>(norm.beta + j);
    float4 w0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), w1 = w0;
    if (to.logits) {                                                     // router: (expert 0, expert 1) of columns j ..
        w0 = *reinterpret_cast<const float4 *>(to.wg + 2 * j);
        w1 = *reinterpret_cast<const float4 *>(to.wg + 2 * j + 4);
    }
    v4i acc = {0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int s = 0; s < NE; ++s)
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, b[p][s]), __builtin_bit_cast(v4i, a[s]), acc, 0, 0, 0);
    const float4 row = make_float4(__builtin_fmaf((float)acc[0], norm.scale, res.x), __builtin_fmaf((float)acc[1], norm.scale, res.y),
                                   __builtin_fmaf((float)acc[2], norm.scale, res.z), __builtin_fmaf((float)acc[3], norm.scale, res.w));
    *reinterpret_cast<float4 *>(rows_s + fr * PITCH + col) = row;
    if (m0 + fr < n_rows) *reinterpret_cast<float4 *>(norm.out + m * E + col) = row;
    __syncthreads();                                                     // and everyone has read its codes, whose place the new ones take
#pragma unroll 1
    for (int r = wave * LANES + lane / LPR; r < kRows; r += WAVES * LANES) {         // wave-uniform: LANES rows each
        const long t = m0 + r;
        const float4 x[1] = {row_or_zero(*reinterpret_cast<const float4 *>(rows_s + r * PITCH + j), in)};
        float mean, rstd, y[4], part[2] = {0.0f, 0.0f};
        row_stats<LPR, 1>(x, l, E, norm.eps, mean, rstd);
        normalise(x[0], mean, rstd, gamma, beta, y);
        if (in) {
            if (t < n_rows) {
                *reinterpret_cast<uint32_t *>(to.codes + t * E + j) = codes_of(y, norm.inv_scale);
                if (to.half)
                    *reinterpret_cast<v4h *>(static_cast<_Float16 *>(to.half) + t * E + j) = v4h{(_Float16)y[0], (_Float16)y[1], (_Float16)y[2], (_Float16)y[3]};
            }
            part[0] = __builtin_fmaf(y[0], w0.x, part[0]);
            part[1] = __builtin_fmaf(y[0], w0.y, part[1]);
            part[0] = __builtin_fmaf(y[1], w0.z, part[0]);
            part[1] = __builtin_fmaf(y[1], w0.w, part[1]);
            part[0] = __builtin_fmaf(y[2], w1.x, part[0]);
            part[1] = __builtin_fmaf(y[2], w1.y, part[1]);
            part[0] = __builtin_fmaf(y[3], w1.z, part[0]);
            part[1] = __builtin_fmaf(y[3], w1.w, part[1]);
        }
        if (to.logits) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float sum = group_sum<LPR>(part[e]);
                if (l == 0 && t < n_rows) to.logits[t * 2 + e] = sum + to.bg[e];
            }
        }
    }
}

template <int NE>
int launch(const int8_t *codes, const NormRows &norm, long T, const NormOut &to, hipStream_t st) {
    linear_norm_kernel<NE><<<dim3((unsigned)((T + kRows - 1) / kRows)), dim3(NE * 256), 0, st>>>(codes, norm, T, to);
    return check_launch("output projection and LayerNorm");
}

}  // namespace

// Every workgroup reads all of Wo, 8 to 72 KB, for 16 rows.  Whole layers with two experts, two launches and one, us:
//   E =  64: 49 rows 28.7, 25.4; 1576 37.0, 33.0; 8192 47.5, 43.5; 25216 64.4, 58.9
//   E = 128: 49 rows 31.6, 29.2; 1576 41.9, 39.3; 12608 70.4, 68.4; 25216 98.4, 100.2
//   E = 192: 49 rows 36.2, 34.6; 1576 49.2, 46.9; 8192 72.5, 69.3; 12608 97.2, 96.5; 25216 134.6, 136.9
//   E = 256 (128 KB): 197 rows 37.9, 39.6; 2364 61.3, 61.2; 8192 84.1, 89.8: not built
bool sa::linear_norm_one_launch(long T, int E) { return (E == 64 || E == 128 || E == 192) && T * E <= 2L << 20; }

int sa::launch_linear_norm(const int8_t *codes, const NormRows &norm, long T, int E, const NormOut &to, hipStream_t st) {
    switch (E) {
        case 64: return launch<1>(codes, norm, T, to, st);
        case 128: return launch<2>(codes, norm, T, to, st);
        case 192: return launch<3>(codes, norm, T, to, st);
    }
    return fail(SA_ERR_UNSUPPORTED, "layer: output projection and LayerNorm of width %d", E);
}
