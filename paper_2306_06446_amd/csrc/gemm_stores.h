// How the accumulators of the two experts' matrix-core layers become output rows (the Store types of gemm_mfma.h).
#pragma once

#include "common.h"
#include "gemm_common.h"

namespace sa {

inline Epilogue with_finite_scale(Epilogue e) {
    e.rq = requant_scale_finite(e.rq);
    return e;
}

template <int MODE>
struct ShiftStore {
    static constexpr int kBytes = (MODE == kEpiRequantLut) ? 1 : 4;
    static constexpr int kTableBytes = (MODE == kEpiRequantLut) ? 256 : 0;
    static constexpr bool kScatter = (MODE == kEpiScatterI32);
    static constexpr bool kLinear = (MODE == kEpiLinearF32 || MODE == kEpiQkvCodes);
    static constexpr bool kSignCodes = (MODE == kEpiQkvCodes);
    static constexpr int kHashBytes = 0;
    Epilogue e;
    void *out;             // int32 rows | int8 hidden rows | scattered fp32 rows
    const void *table;     // the 256-entry activation table
    const float *gate;
    bool accumulate;
    size_t out_block;
    float *parts[3];       // kEpiLinearF32: column blocks, residual and scale
    int part_width;
    const float *residual;
    float scale;
    uint64_t *codes[2];    // kEpiQkvCodes: sign codes of column blocks 0 and 1
    int code_cols, head_dim, tokens, heads;
    explicit ShiftStore(const Epilogue &epi)     // epi.rq is made finite here: convert() relies on it
        : e(with_finite_scale(epi)),
          out(MODE == kEpiInt32 ? (void *)epi.y : MODE == kEpiRequantLut ? (void *)epi.h
              : MODE == kEpiLinearF32 ? (void *)epi.parts[0] : MODE == kEpiQkvCodes ? (void *)epi.parts[2] : (void *)epi.yf),
          table(epi.lut),
          gate(MODE == kEpiScatterI32 ? epi.gate : nullptr),
          accumulate(MODE == kEpiScatterI32 && epi.accumulate),
          out_block(epi.h_block),
          parts{epi.parts[0], epi.parts[1], epi.parts[2]},
          part_width(epi.part_width > 0 ? epi.part_width : 4),
          residual(epi.residual),
          scale(epi.lin_scale),
          codes{epi.codes[0], epi.codes[1]},
          code_cols(MODE == kEpiQkvCodes ? 2 * epi.part_width : 0),
          head_dim(epi.head_dim > 0 ? epi.head_dim : 64),
          tokens(epi.tokens > 0 ? epi.tokens : 1),
          heads(epi.heads) {}
    __device__ inline uint32_t convert(int32_t acc, int n, const uint8_t *lds_table) const {
        if (MODE == kEpiInt32) return (uint32_t)(acc + (e.bias ? e.bias[n] : 0));
        if (MODE == kEpiRequantLut) return lds_table[requant_index(acc, e.rq)];
        if (MODE == kEpiLinearF32 || MODE == kEpiQkvCodes) return __builtin_bit_cast(uint32_t, (float)acc);   // scaled at the store
        return __builtin_bit_cast(uint32_t, e.out_scale * (float)acc);
    }
};

// a * Phi(a) = max(a, 0) - |a| * Phi(-|a|), with Phi(-x) = exp(-x^2 / 2) * t * P(t), t = 1 / (1 + 0.35 x): the form of
// Hastings' approximations of erf, P fitted here (least squares in the relative error, reweighted towards the minimax one) to
// 2.6e-7.  No 1 + erf that cancels for negative a: within 1e-3 of the last bit of the fp16 result everywhere, where
// 0.5 a (1 + erff) was off by up to 1.7 of them; and no branches: erff takes both of its two in almost every wavefront, which
// was 8 us of every 192 x 128 tile's way out with two workgroups to a CU (12608 x 768 tokens through a layer 370 -> 362 us).
__device__ inline float gelu_erf(float a) {
    const float x = __builtin_fminf(__builtin_fabsf(a), 20.0f);       // finite: Inf * 0 below would be NaN
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.35f, x, 1.0f));
    float p = 0.047504745f;
    p = __builtin_fmaf(p, t, -0.195814105f);
    p = __builtin_fmaf(p, t, 0.22912737f);
    p = __builtin_fmaf(p, t, -0.0057044461f);
    p = __builtin_fmaf(p, t, 0.14950726f);
    p = __builtin_fmaf(p, t, 0.13548473f);
    p = __builtin_fmaf(p, t, 0.13989458f);
    const float tail = x * __builtin_amdgcn_exp2f(x * x * -0.72134752f) * t;      // exp(-x^2 / 2) in powers of two
    return __builtin_fmaf(-tail, p, __builtin_fmaf(0.5f, __builtin_fabsf(a), 0.5f * a));
}

template <int MODE>
struct MultStore {
    static constexpr int kBytes = (MODE == kEpiGeluHalf) ? 2 : 4;
    static constexpr int kTableBytes = 0;
    static constexpr bool kScatter = (MODE == kEpiScatterF32);
    static constexpr bool kLinear = false;
    static constexpr bool kSignCodes = false;
    static constexpr int kHashBytes = 0;
    void *out;                      // compact fp32 rows | fp16 hidden rows | scattered fp32 rows
    const void *table = nullptr;
    const float *gate;
    bool accumulate;
    size_t out_block;
    explicit MultStore(const Epilogue &epi)
        : out(MODE == kEpiFloat ? (void *)epi.of : MODE == kEpiGeluHalf ? (void *)epi.hh : (void *)epi.yf),
          gate(MODE == kEpiScatterF32 ? epi.gate : nullptr),
          accumulate(MODE == kEpiScatterF32 && epi.accumulate),
          out_block(epi.h_block) {}
    __device__ inline uint32_t convert(float a, int, const uint8_t *) const {
        if (MODE == kEpiGeluHalf) return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)gelu_erf(a));
        return __builtin_bit_cast(uint32_t, a);
    }
};

}  // namespace sa
