// What the three kernels that hash rows on the matrix cores share (binarize_mfma.hip, norm_hash.hip, linear_hash.hip): where code words lie,
// the fp16 terms of an operand, and the defining chain for what the products leave open.
#pragma once

#include "common.h"
#include "hash_margin.h"

namespace sa {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct RowMap {
    FastDiv by_h, by_n;
    int N, H, W;
    __device__ inline size_t row_words(uint32_t row) const {     // first code word of a row of the flattened input
        const uint32_t t = by_h(row), h = row - t * (uint32_t)H, b = by_n(t), n = t - b * (uint32_t)N;
        return ((size_t)(b * (uint32_t)H + h) * N + n) * W;
    }
};

// Up to two tensors of the same shape are hashed by one launch (Q and K of a block).
struct Tensors {
    const float *x0, *x1;
    uint64_t *codes0, *codes1;
};

// (a, b) as fp16 terms, a in the lower half: upper terms, and what they leave.
__device__ inline void split_f16_pair(float a, float b, uint32_t &upper, uint32_t &lower) {
    const v2f x = {a, b};
    const v2h h = __builtin_convertvector(x, v2h);
    upper = __builtin_bit_cast(uint32_t, h);
    v2f r;                                        // a - h[0], b - h[1]: exact, one operation each that reads its half of h itself
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r[0]) : "v"(upper), "v"(a));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r[1]) : "v"(upper), "v"(b));
    lower = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, v2h));
}

// Zeros.  Of a row of zeros, whose token may be padding, every sum of the chain is 0 and every bit set, unless a column has infinities or
// NaN; of a column of zeros every bit of finite rows.  The products give 0 there, whose sign is right, and the kernels that hash in the
// projection, whose chain takes its columns from memory, keep it.  Layers with a tenth of the rows of zeros, us, hash a launch of its own /
// in the projection with the chain for them / so: 16384 x 256, 256 bits 390, 1148, 128; 12608 x 768, 128 bits 590, 832, 292; 197 x 192 51, 35, 29
// (of other rows 0.2 to 0.4 % longer).
// Whether |x|^2 = 0 says that a row is all zeros: its elements are integers times scale, whose squares then do not underflow.
__device__ inline bool scale_is_exact(float scale) { return __builtin_fabsf(scale) >= 0x1p-60f; }
// n2, a thread's share of a column's |r|^2, for the same: 0 only where its elements x are zeros.
template <int N>
__device__ inline float column_norm(float n2, const float (&x)[N][8]) {
    if (n2 == 0.0f) {
        uint32_t some = 0;
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) some |= __builtin_bit_cast(uint32_t, x[i][e]) << 1;
        if (some != 0) n2 = 0x1p-126f;
    }
    return n2;
}

// A bit whose sign the products leave open: row of the flattened input, column, the bit as stored, which tensor.
__device__ inline uint64_t open_bit(uint32_t row, int col, uint32_t bit, bool second) {
    return (uint64_t)row | ((uint64_t)col << 32) | ((uint64_t)bit << 48) | ((uint64_t)second << 49);
}

// Re-runs the defining chain for one such bit and flips it where the pre-pass had it wrong.  cols: hash columns from c_first on, fp32,
// `pitch` from one row of the hash matrix to the next.  RND steps of the chain per round trip of loads.
template <int D, int RND>
__device__ inline void settle_entry(uint64_t e, const Tensors &ts, const float *cols, int pitch, int c_first, const RowMap &map) {
    const uint32_t row = (uint32_t)e;
    const int col = (int)((e >> 32) & 0xffffu);
    const bool prov = (e >> 48) & 1u;
    const bool second = (e >> 49) & 1u;
    const float *xr = (second ? ts.x1 : ts.x0) + (size_t)row * D;
    uint64_t *codes = second ? ts.codes1 : ts.codes0;
    float acc = 0.0f;
    // loads first, then the fmas in their defined order
#pragma unroll 1
    for (int k0 = 0; k0 < D; k0 += RND) {
        float xv[RND];
#pragma unroll
        for (int q = 0; q < RND / 4; ++q) {
            const float4 t4 = *reinterpret_cast<const float4 *>(xr + k0 + 4 * q);
            xv[4 * q] = t4.x; xv[4 * q + 1] = t4.y; xv[4 * q + 2] = t4.z; xv[4 * q + 3] = t4.w;
        }
#pragma unroll
        for (int k = 0; k < RND; ++k) acc = __builtin_fmaf(xv[k], cols[(k0 + k) * pitch + col - c_first], acc);
    }
    const bool exact = acc >= 0.0f;
    if (exact != prov)
        atomicXor(reinterpret_cast<unsigned long long *>(codes + map.row_words(row) + (col >> 6)), 1ull << (col & 63));
}

}  // namespace sa
