// Internal helpers of libshiftadd (host-side validation, error text, launch checks).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "shiftadd.h"

namespace sa {

// Records a message for sa_last_error() and returns `code`.
int fail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool aligned4(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

// Turns the status of the launch just issued into an SA code.
int check_launch(const char *what);

// Zero-fills `bytes` (a multiple of 4) with a kernel (safe under graph capture).
int launch_zero(void *p, size_t bytes, hipStream_t st);

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

constexpr int kWave = 64;

// n / d for 0 <= n < 2^31 as one multiplication and one shift.
struct FastDiv {
    uint32_t mul;
    int shift;
    explicit FastDiv(uint32_t d) {
        int s = 0;
        while ((1ull << s) < d) ++s;
        shift = 31 + s;
        mul = (uint32_t)(((1ull << shift) + d - 1) / d);
    }
    __host__ __device__ inline uint32_t operator()(uint32_t n) const { return (uint32_t)(((uint64_t)n * mul) >> shift); }
};

// Resolves an sa_rows descriptor inside a kernel (all lanes get the same values).
struct RowSel {
    const int32_t *rows;    // may be null: identity
    const int32_t *counts;  // may be null: n_rows = max_rows
    int expert;
    long max_rows;
};

__device__ inline void resolve_rows(const RowSel &sel, const int32_t *&rows, long &n_rows) {
    rows = sel.rows;
    n_rows = sel.max_rows;
    if (sel.counts != nullptr) {
        long off = 0;
        for (int e = 0; e < sel.expert; ++e) off += sel.counts[e];
        long cnt = sel.counts[sel.expert];
        rows = sel.rows + off;
        n_rows = cnt < sel.max_rows ? cnt : sel.max_rows;
    }
}

int validate_rows(const sa_rows *rows, RowSel *out);

// The argument checks of the entry points that sa_block_forward and sa_layer_forward are made of, apart from their launches:
// both call all of them first, so that a call that is refused has launched nothing.  Each is that entry point's whole validation;
// sizes of zero pass.
int check_binarize(const float *x, int B, int N, int H, int d, const float *proj, int nbits, const uint64_t *codes, int variant);
int check_binarize_pair(const float *q, const float *k, int B, int N, int H, int d, const float *proj, int nbits,
                        const uint64_t *q_codes, const uint64_t *k_codes);
int check_additive_attention(const uint64_t *q_codes, const uint64_t *k_codes, const float *v, const float *out, int B, int H, int Nq,
                             int Nk, int nbits, int dv, const float *kv, int phases, const void *workspace, size_t workspace_bytes);
int check_hamming_attention(const uint64_t *q_codes, const uint64_t *k_codes, const float *v, const float *out, int B, int H, int Nq,
                            int Nk, int nbits, int dv, float scale, const int16_t *scores_or_null, const int8_t *xq_or_null,
                            const void *xh_or_null, int variant);
int check_layernorm(const float *x, long T, int E, const float *gamma, const float *beta, const float *ln_or_null,
                    const int8_t *q_or_null, const void *xh_or_null, const float *wg_or_null, const float *bg_or_null, int n_experts,
                    const float *logits_or_null);
int check_shift_linear_f32(const int8_t *x, const uint8_t *w4, long M, int K, int N, int variant, const float *residual_or_null,
                           int parts, const float *y0, const float *y1, const float *y2, const void *workspace, size_t workspace_bytes);
int check_shift_linear_qkv_codes(const int8_t *x, const uint8_t *wqkv, int B, int N, int H, int E, int variant, float scale,
                                 const uint64_t *q_codes, const uint64_t *k_codes, const float *v, const void *workspace,
                                 size_t workspace_bytes);
int check_moe_dispatch(const float *logits, long T, int E, int32_t *perm, int32_t *expert_of, int32_t *counts, float *gate,
                       const void *workspace, size_t workspace_bytes);
int check_shift_mlp(const int8_t *xq, const sa_rows *rows, RowSel *sel, int E, int hid, const uint8_t *w1, const uint8_t *w2,
                    const int8_t *lut, const int32_t *y2_or_null, const float *y_or_null, const float *gate_or_null, int variant,
                    int stages, const void *workspace, size_t workspace_bytes);
bool shift_rows_fit(long rows, int variant);         // rows of one launch of a Shift layer

// 16 bytes to memory past the caches' reuse order: for 32-bit outputs, which are large and written once, and otherwise push out
// the operands of the launch that writes them.  12608 x 1536 <- 384 and back, int32: 72 -> 60 us; the layers with fp32 outputs of
// 12608 x 768 tokens 0 to 4 us each; Q(K^T V) at 8 x 4 x 16384 x 256 bits x 64 70 -> 64 us.  It pays even where the next
// launch reads them again, as Q, K, V and y of a layer: 12608 x 768 tokens 341 -> 333 us, 25088 x 64 63.0 -> 60.0, 16384 x
// 256 128.4 -> 127.4; one image of 197 x 192, which fits the L2, 42.6 -> 43.0.  For the narrow outputs that the next kernel
// reads it gained nothing, for the reads of Q and K it lost (pvt-sized attention 28.8 -> 30.5 us).
__device__ inline void store_streaming(void *dst, const uint4 &v) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(u4{v.x, v.y, v.z, v.w}, reinterpret_cast<u4 *>(dst));
}

// One wavefront-wide direct global -> LDS load, no registers and nothing for the compiler to wait for: lane l's 16 (4)
// bytes at `src` land at LDS byte lds_base + 16 (4) * l (lds_base is the same in every lane).
__device__ inline void direct_load_16(const void *src, uint32_t lds_base) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off\n\t"
        :
        : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(src)
        : "memory");
}
// The same with the address as a wavefront-uniform base and a 32-bit offset per lane (no vector address arithmetic).
__device__ inline void direct_load_16(const void *base, uint32_t lane_off, uint32_t lds_base) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2\n\t"
        :
        : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(lane_off), "s"(base)
        : "memory");
}
__device__ inline void direct_load_4(const void *base, uint32_t lane_off, uint32_t lds_base) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dword %1, %2\n\t"
        :
        : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(lane_off), "s"(base)
        : "memory");
}
__device__ inline void direct_load_4(const void *src, uint32_t lds_base) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dword %1, off\n\t"
        :
        : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(src)
        : "memory");
}

// The waits that kernels place by hand, for what the compiler does not track (direct loads) or is not meant to wait for.  To the
// compiler the builtin alone is no memory access: it may move a read of what a direct load brought to before it, or a store to
// behind it.  The empty statements keep memory accesses on their sides.
//   wait_loads_in_flight<N> : until at most N of this wavefront's vector-memory operations are still in flight (loads complete
//                             in issue order, so the oldest ones are the ones that have landed; stores count too)
//   wait_lds_reads          : until this wavefront's LDS operations are done
template <int N>
__device__ inline void wait_loads_in_flight() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
    asm volatile("" ::: "memory");
}
__device__ inline void wait_lds_reads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("" ::: "memory");
}

// One Linear layer on the rows an expert was given, gated and scattered (the two experts of sa_moe_linear):
//   y[rows[i], :] = gate[rows[i]] * (xh[rows[i], :] . W^T)                      fp16 operands   (mult_mlp.hip)
//   y[rows[i], :] = gate[rows[i]] * out_scale * (xq[rows[i], :] . Wshift^T)      int8 / 4-bit    (shift_linear.hip)
// Arguments are checked by the caller; `planes` is shift_linear_rows_workspace_bytes(K, N, variant) bytes.
int mult_linear_rows(const void *xh_all, const RowSel &sel, int K, int N, const void *w_f16, float *y, const float *gate,
                     hipStream_t st);
size_t shift_linear_rows_workspace_bytes(int K, int N, int variant);
int shift_linear_rows(const int8_t *xq_all, const RowSel &sel, int K, int N, const uint8_t *w4, float out_scale, float *y,
                      const float *gate, int variant, void *planes, hipStream_t st);
// Small jobs that can ride in another kernel's launch (side_work.h).
constexpr int kMaxExperts = 8;
constexpr long kSideRouteTokens = 32768;     // the one-launch routing takes up to this many tokens
struct RouteWork {                           // sa_moe_dispatch in one launch
    const float *logits = nullptr;
    long T = 0;                              // 0: none
    int E = 2;
    int32_t *expert_of = nullptr;
    float *gate = nullptr;
    int32_t *counts = nullptr, *perm = nullptr;
};
struct DecodeWork {                          // packed weights [N, K], K a multiple of 64, to their two planes
    const uint4 *w4[3] = {nullptr, nullptr, nullptr};
    uint4 *plane_a[3] = {nullptr, nullptr, nullptr}, *plane_b[3] = {nullptr, nullptr, nullptr};
    long chunks[3] = {0, 0, 0};              // of 32 weights; 0: none
};
struct ZeroWork {                            // words to be cleared for a later launch, by the first workgroup of this one
    uint32_t *words = nullptr;
    int n = 0;
};
struct SideWork {
    RouteWork route;
    DecodeWork decode;
    ZeroWork zero;
    bool any() const { return route.T > 0 || decode.chunks[0] > 0 || zero.n > 0; }
};
__device__ inline void zero_words(const ZeroWork &z) {
    for (int i = threadIdx.x; i < z.n; i += blockDim.x) z.words[i] = 0u;
}
void add_decode(DecodeWork *w, const uint8_t *w4, int K, int N, void *planes);
// Both layers of an MLP; `workspace` as sa_shift_mlp lays it out.  The planes then are what the prepared variant takes.
void shift_mlp_decode(DecodeWork *w, const uint8_t *w1, const uint8_t *w2, int E, int hid, long max_rows, void *workspace,
                      const uint8_t **planes1, const uint8_t **planes2);
int launch_decode_work(const DecodeWork &w, hipStream_t st);
int launch_decode_work(const DecodeWork &w, const DecodeWork &w2, hipStream_t st);      // both in one launch
// The decoded planes of one layer: the caller's (prepared variant) or `planes`, filled by this call.
int shift_linear_planes(const uint8_t *w4, int K, int N, int variant, void *planes, hipStream_t st, const int8_t **out);

// Shift and Mult expert side by side in one launch per layer, matrix cores only (experts.hip).  The rows of the two
// selections add up to at most max_rows, which is the same in both; every token belongs to one of them.
struct ExpertPair {
    const int8_t *xq;        // int8 codes and fp16 rows of every token
    const void *xh;
    RowSel shift_rows, mult_rows;
    float *y;                // [T, N]: scattered, gated
    const float *gate;
    float out_scale;         // of the Shift expert
};
int expert_pair_mlp(const ExpertPair &p, int E, int hid, const int8_t *w1_planes, const int8_t *w2_planes, const void *mw1,
                    const void *mw2, float requant_scale, const int8_t *lut, bool accumulate, int8_t *shift_hidden,
                    void *mult_hidden, hipStream_t st);
int expert_pair_linear(const ExpertPair &p, int K, int N, const int8_t *w_planes, const void *w_f16, hipStream_t st);
// Both layers of a Shift MLP in one launch, on decoded planes (shift_mlp.hip): whether it takes the shape, and the launch.
// out: yf, gate, out_scale, accumulate.
struct Epilogue;
enum MlpCall { kMlpPacked, kMlpPrepared, kMlpInLayer };      // weights still to be decoded; decoded; the same, rows not normalised yet
bool shift_mlp_one_launch(const RowSel &sel, int E, int hid, MlpCall call);
// fp32 rows [max_rows, E] whose LayerNorm, as int8 codes (static scale), an MLP takes: x, or, with wo (decoded planes [E, E]),
// out = residual + scale * wo . codes, which the launch leaves there as well.
struct NormRows {
    const float *x = nullptr, *gamma = nullptr, *beta = nullptr;
    float eps = 0.0f, inv_scale = 1.0f;
    const int8_t *wo = nullptr;
    const float *residual = nullptr;
    float scale = 1.0f, *out = nullptr;
    ZeroWork zero;           // (launch_norm_linear, launch_norm_hash)
};
// Of the rows x; of all rows of norm, or of those it makes of the codes x (they may be the output's: a workgroup reads its rows
// before it writes them).
int launch_shift_mlp(const int8_t *x, const NormRows *norm, const RowSel &sel, int E, int hid, const int8_t *w1_planes,
                     const int8_t *w2_planes, const int8_t *lut, float requant_scale, const Epilogue &out, hipStream_t st);
// norm.out = norm.residual + norm.scale * norm.wo . codes and its LayerNorm in one launch (linear_norm.hip): whether it is the faster way,
// and the launch.  The new codes may take the old ones' place.
struct NormOut {
    int8_t *codes;
    void *half;              // fp16 rows, or null
    const float *wg, *bg;    // router of two experts [E, 2], [2]
    float *logits;           // [T, 2], or null
};
bool linear_norm_one_launch(long T, int E);
int launch_linear_norm(const int8_t *codes, const NormRows &norm, long T, int E, const NormOut &to, hipStream_t st);
// The whole MLP half of a layer, or the MLP of a block, in one launch for few rows (few_rows_mlp.hip): the workspace it takes (none: it
// does not take the shape, or has no gain by it), of which the first ticket_bytes are zero before the launch; and the launch.
struct FewRowsPlan {
    size_t bytes = 0, ticket_bytes = 0;
    int mi = 1;              // 16-row tiles of a workgroup
};
struct FewRowsMlp {
    const int8_t *codes;     // of the attention's output (layer), of the rows (block)
    const void *half;        // block with a Mult expert: the rows as fp16
    const NormRows *norm;    // layer: residual, scale, wo, LayerNorm; else null
    const float *wg, *bg;    // layer with two experts: the router
    const float *logits;     // block with two experts: [T, 2]
    long T;
    int E, hid;
    const int8_t *w1, *w2, *lut;     // decoded planes
    const void *mw1, *mw2;   // Mult expert, or null
    float requant_scale, out_scale;
    float *y;                // layer: residual + ..., complete
    void *workspace;
};
FewRowsPlan plan_few_rows(long T, int E, int hid, bool moe, bool layer);
int launch_few_rows(const FewRowsMlp &m, const FewRowsPlan &p, hipStream_t st);
// sa_layernorm_quant without its argument checks; `zero` is cleared by its first workgroup.
int launch_layernorm(const float *x, long T, int E, const float *gamma, const float *beta, float eps, float inv_scale, float *ln, int8_t *q,
                     void *xh, const float *wg, const float *bg, int n_experts, float *logits, const ZeroWork &zero, hipStream_t st);
// LayerNorm of all T rows of norm.x and the Q, K, V projection of its codes (decoded planes [3E, E]) in one launch
// (norm_linear.hip): whether it is the faster way, and the launch.
bool norm_linear_one_launch(long T, int E);
int launch_norm_linear(const NormRows &norm, long T, int E, const int8_t *wqkv_planes, float scale, float *q, float *k, float *v,
                       hipStream_t st);
// The same with the hash of Q and K behind it (norm_hash.hip): Q and K leave as code words, and in q and k only the rows that the hash
// asks its defining chain about.
bool norm_hash_one_launch(long T, int E, int H, int nbits);
int launch_norm_hash(const NormRows &norm, int B, int N, int H, int E, const int8_t *wqkv_planes, float scale, const float *proj, int nbits,
                     float *q, float *k, uint64_t *q_codes, uint64_t *k_codes, float *v, hipStream_t st);
// The projection of codes that are normalised already, with the hash of Q and K in it (linear_hash.hip).
bool linear_hash_one_launch(long T, int E, int H, int nbits, bool packed);
int launch_linear_hash(const int8_t *codes, int B, int N, int H, int E, const int8_t *wqkv_planes, float scale, const float *proj, int nbits,
                       float *q, float *k, uint64_t *q_codes, uint64_t *k_codes, float *v, hipStream_t st);
// The routing of sa_moe_dispatch without its argument checks (moe.hip).
size_t moe_dispatch_scratch_bytes(long T, int E);
int moe_dispatch_launch(const float *logits, long T, int E, int32_t *perm, int32_t *expert_of, int32_t *counts, float *gate,
                        void *scratch, hipStream_t st);

// Hash pre-pass on the matrix cores with exact fallback (binarize_mfma.hip).
bool binarize_mfma_supported(int d, int nbits);
int launch_binarize_mfma(const float *x0, const float *x1_or_null, const float *proj, uint64_t *codes0,
                         uint64_t *codes1_or_null, long rows, int N, int H, int d, int nbits, hipStream_t st,
                         const SideWork &side = SideWork());
// sa_binarize_pair without proj, without its argument checks: a launch each; `zero` is cleared by the first.
int launch_sign_pair(const float *q, const float *k, long rows, int N, int H, int d, uint64_t *q_codes, uint64_t *k_codes,
                     const ZeroWork &zero, hipStream_t st);
// Whether sa_binarize_pair runs that kernel for these operands, in one launch (binarize.hip).
bool binarize_pair_one_launch(const float *q, const float *k, const float *proj, const uint64_t *q_codes, const uint64_t *k_codes,
                              long rows, int d, int nbits);

// Additive attention on the matrix cores (additive_mfma.hip).
struct AdditiveMfmaPlan {
    int groups;             // groups of up to 4 code words
    int splits;             // token ranges (partial K^T V each)
    int tokens_per_block;
};
// What Q(K^T V) reads and leaves.  kv_in: [splits][B*H][nbits][dv] partials of K^T V, summed in ascending order (splits
// = 1: K^T V itself); kv_out (or null): the sum.  ksum_in / ksum_out: the same for the bit counts of {0,1} codes, int32
// [splits][B*H][nbits].  Rows leave as scale * acc, or acc / (normaliser + eps) with {0,1} codes, in any of three forms:
// fp32, the int8 codes of the activation quantiser, fp16.
struct AddFused {
    const float *kv_in = nullptr;
    float *kv_out = nullptr;
    const int32_t *ksum_in = nullptr;
    int32_t *ksum_out = nullptr;
    int splits = 1;
    float scale = 1.0f, eps = 0.0f;
    float *out = nullptr;
    int8_t *xq = nullptr;
    _Float16 *xh = nullptr;
    float act_inv_scale = 0.0f;
    bool keep = false;       // {0,1} codes: the outputs stay in the caches for who reads them next
    bool rows_ahead = false; // (launch_qkv_mfma) the addresses of a tile's rows are made before the first one leaves
};
bool additive_mfma_ktv_supported(int nbits, int dv);
bool additive_mfma_qkv_supported(int nbits, int dv);
bool additive_mfma_sums_partials(int splits, int nbits, int dv);
AdditiveMfmaPlan plan_additive_mfma(int B, int H, int Nk, int nbits, int dv);
// zero_one: a clear code bit stands for 0 instead of -1, and the bit counts of the range are left in ksum.
int launch_ktv_mfma(const uint64_t *k_codes, const float *v, float *dst, int32_t *ksum, int B, int H, int Nk, int nbits, int dv,
                    const AdditiveMfmaPlan &p, bool zero_one, hipStream_t st);
int launch_ktv_sum(const float *part, float *kv, const int32_t *ksum_part, int32_t *ksum, long BH, int nbits, int dv, int splits,
                   hipStream_t st);
// Short sequences, +-1 codes: both in one launch.
bool additive_mfma_one_launch(const AdditiveMfmaPlan &p, int Nq, int Nk, int nbits);
int launch_ktv_qkv(const uint64_t *k_codes, const float *v, float *kv, const uint64_t *q_codes, const AddFused &f, int B, int H,
                   int Nq, int Nk, int nbits, int dv, hipStream_t st);
int launch_qkv_mfma(const uint64_t *q_codes, const AddFused &f, int B, int H, int Nq, int nbits, int dv, bool zero_one,
                    hipStream_t st);
// sa_additive_attention (both phases) whose output also leaves as the int8 codes (and fp16 rounding) the MLP reads, from
// the kernel that computes it.  `out` is always a valid buffer; want_out = false: nothing but those forms is read.
int additive_attention_fused(const uint64_t *q_codes, const uint64_t *k_codes, const float *v, float *out, bool want_out,
                             int B, int H, int N, int nbits, int dv, float scale, float *kv, int8_t *xq, _Float16 *xh,
                             float act_inv_scale, void *workspace, size_t workspace_bytes, void *stream);

}  // namespace sa

#define SA_REQUIRE(cond, code, ...) \
    do {                            \
        if (!(cond)) return ::sa::fail((code), __VA_ARGS__); \
    } while (0)
