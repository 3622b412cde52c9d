// Two small jobs that nothing before the experts waits for, as device code that any launch can carry along: the routing of
// two-expert tokens and the decode of 4-bit shift weights into int8 planes.  As launches of their own they cost 3 to 7 us
// each, mostly launch latency on a chip that is nearly idle.
#pragma once

#include "common.h"

namespace sa {

__device__ inline uint64_t lanemask_lt(int lane) { return (lane == 0) ? 0ull : (~0ull >> (64 - lane)); }

// The index of the largest logit of token t (the first one among equals).
__device__ inline int top1(const float *__restrict__ l, int E) {
    int best = 0;
    float lb = l[0];
    for (int e = 1; e < E; ++e) {
        const float le = l[e];
        if (le > lb) { lb = le; best = e; }
    }
    return best;
}

// One launch for the whole dispatch: workgroup b of kOneTok threads owns tokens [kOneTok b, kOneTok (b + 1)).  Pass 1 over all T tokens
// (thread i takes tokens i, i + kOneTok, ...; the loads of a thread are independent and issued together): per expert, how
// many tokens it gets in all and how many of them lie in workgroups before b.  Pass 2: the workgroup's own tokens,
// ranked by ballot / popcount behind those counts.
template <int kOneTok, int E_FIXED>
__device__ __forceinline__ void route_scatter_block(const RouteWork &w, int block) {
    const float *__restrict__ logits = w.logits;
    const long T = w.T;
    const int E_runtime = w.E;
    int32_t *__restrict__ expert_of = w.expert_of, *__restrict__ counts = w.counts, *__restrict__ perm = w.perm;
    float *__restrict__ gate = w.gate;
    const int E = E_FIXED > 0 ? E_FIXED : E_runtime;
    constexpr int kWaves = kOneTok / 64;
    __shared__ int32_t wave_cnt[kWaves][kMaxExperts];
    __shared__ int32_t red[kWaves][2 * kMaxExperts];
    __shared__ int32_t base_s[kMaxExperts];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long first = (long)block * kOneTok;              // tokens before `first` belong to earlier workgroups
    int below[kMaxExperts], all[kMaxExperts];
#pragma unroll
    for (int e = 0; e < kMaxExperts; ++e) below[e] = all[e] = 0;
    float2 own = make_float2(0.0f, 0.0f);                       // E == 2: the logits of this thread's own token, met in pass 1
    if (E_FIXED == 2) {
        const float2 *l2 = reinterpret_cast<const float2 *>(logits);
        constexpr int kBatch = 16;                              // independent loads in flight per thread: kBatch * kOneTok tokens per round trip
        for (long t0 = tid; t0 < T; t0 += (long)kBatch * kOneTok) {
            float2 l[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const long t = t0 + (long)i * kOneTok;
                l[i] = t < T ? l2[t] : make_float2(0.0f, 0.0f);
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const long t = t0 + (long)i * kOneTok;
                const int one = (t < T && l[i].y > l[i].x) ? 1 : 0;     // expert 1 only if strictly larger
                all[1] += one;
                below[1] += t < first ? one : 0;
                if (t == first + tid) own = l[i];
            }
        }
        const int mine_all = T > tid ? (int)((T - tid + kOneTok - 1) / kOneTok) : 0;    // tokens this thread looked at
        const long fb = first - tid;
        const int mine_below = fb > 0 ? (int)((fb + kOneTok - 1) / kOneTok) : 0;          // ... and those before `first`
        all[0] = mine_all - all[1];
        below[0] = mine_below - below[1];
    } else {
        for (long t = tid; t < T; t += kOneTok) {
            const int best = top1(logits + (size_t)t * E, E);
#pragma unroll
            for (int e = 0; e < kMaxExperts; ++e) {
                all[e] += best == e ? 1 : 0;
                below[e] += (best == e && t < first) ? 1 : 0;
            }
        }
    }
#pragma unroll
    for (int e = 0; e < kMaxExperts; ++e) {
        if (e >= E) continue;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            below[e] += __shfl_xor(below[e], off, 64);
            all[e] += __shfl_xor(all[e], off, 64);
        }
        if (lane == 0) { red[wave][e] = below[e]; red[wave][kMaxExperts + e] = all[e]; }
    }
    __syncthreads();
    if (tid < E) {
        int bl = 0, al = 0;
        for (int w = 0; w < kWaves; ++w) { bl += red[w][tid]; al += red[w][kMaxExperts + tid]; }
        red[0][tid] = bl;                       // (row 0 of red has been read by this thread only)
        red[0][kMaxExperts + tid] = al;
    }
    __syncthreads();
    if (tid == 0) {
        int start = 0;
        for (int e = 0; e < E; ++e) {
            base_s[e] = start + red[0][e];
            if (block == 0) counts[e] = red[0][kMaxExperts + e];
            start += red[0][kMaxExperts + e];
        }
    }
    const long t = first + tid;
    int mine = -1;
    if (t < T) {
        if (E_FIXED == 2) {
            mine = own.y > own.x ? 1 : 0;
            const float lb = mine ? own.y : own.x;
            const float den = __expf(own.x - lb) + __expf(own.y - lb);      // the same sum, in the same order, as the general path
            expert_of[t] = mine;
            gate[t] = 1.0f / den;
        } else {
            const float *l = logits + (size_t)t * E;
            mine = top1(l, E);
            const float lb = l[mine];
            float den = 0.0f;
            for (int e = 0; e < E; ++e) den += __expf(l[e] - lb);
            expert_of[t] = mine;
            gate[t] = 1.0f / den;
        }
    }
    int rank = 0;
    for (int e = 0; e < E; ++e) {
        const uint64_t m = __ballot(mine == e);
        if (mine == e) rank = __builtin_popcountll(m & lanemask_lt(lane));
        if (lane == 0) wave_cnt[wave][e] = __builtin_popcountll(m);
    }
    __syncthreads();
    if (mine >= 0) {
        int before = 0;
        for (int w = 0; w < wave; ++w) before += wave_cnt[w][mine];
        perm[base_s[mine] + before + rank] = (int32_t)t;
    }
}

// 8 nibbles of `x` (k ascending from bit 0) -> 8 int8 of plane A and 8 of plane B, k order.
__device__ inline void decode8(uint32_t x, uint32_t outA[2], uint32_t outB[2]) {
    // magnitude tables indexed by e: bytes 0..3 in the low word, 4..7 in the high word
    constexpr uint32_t TA_LO = 0x08040201u, TA_HI = 0x40402010u;   // 1 2 4 8 | 16 32 64 64
    constexpr uint32_t TB_LO = 0x00000000u, TB_HI = 0x40000000u;   // 0 .. 0 64
    const uint32_t nibs[2] = {x & 0x0F0F0F0Fu, (x >> 4) & 0x0F0F0F0Fu};   // even k, odd k
    uint32_t a[2], b[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const uint32_t sel = nibs[p] & 0x07070707u;
        const uint32_t s1 = (nibs[p] >> 3) & 0x01010101u;          // 1 where negative
        const uint32_t m = s1 * 0xFFu;                             // 0xFF where negative
        const uint32_t pa = __builtin_amdgcn_perm(TA_HI, TA_LO, sel);
        const uint32_t pb = __builtin_amdgcn_perm(TB_HI, TB_LO, sel);
        a[p] = (pa ^ m) + s1;                 // per byte: ~pa + 1 = -pa (pa >= 1: no carry)
        b[p] = pb | (m & (pb << 1));          // 0x40 -> 0xC0 = -64 where negative
    }
    // interleave even / odd back into k order: k0 k1 k2 k3 | k4 k5 k6 k7
    outA[0] = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u);
    outA[1] = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);
    outB[0] = __builtin_amdgcn_perm(b[1], b[0], 0x05010400u);
    outB[1] = __builtin_amdgcn_perm(b[1], b[0], 0x07030602u);
}

// Workgroups of THREADS threads that a DecodeWork takes, a chunk (32 weights, 16 bytes in, 32 bytes out to each plane) to a thread.
template <int THREADS>
__host__ __device__ inline long decode_blocks(const DecodeWork &w) {
    long n = 0;
    for (int m = 0; m < 3; ++m) n += (w.chunks[m] + THREADS - 1) / THREADS;
    return n;
}
// A workgroup has one matrix, so what is read of the kernel's arguments is the same in all lanes.  (Chosen by each lane, the compiler kept
// a copy of the arguments in scratch memory, written and read by every thread: 768 x 3072 and 3072 x 768 weights took 9.8 us
// in a launch of their own and 16.8 with 768 x 2304 ones; 5.7 and 6.4 so.)
template <int THREADS>
__device__ __forceinline__ void decode_block(const DecodeWork &w, long block) {
    const uint4 *w4 = w.w4[0];
    uint4 *pa = w.plane_a[0], *pb = w.plane_b[0];
    long chunks = w.chunks[0];
#pragma unroll
    for (int m = 1; m < 3; ++m) {
        const long blocks = (chunks + THREADS - 1) / THREADS;
        if (block < blocks) break;
        block -= blocks;
        w4 = w.w4[m];
        pa = w.plane_a[m];
        pb = w.plane_b[m];
        chunks = w.chunks[m];
    }
    const long i = block * THREADS + threadIdx.x;
    if (i >= chunks) return;
    const uint4 wv = w4[i];
    const uint32_t wd[4] = {wv.x, wv.y, wv.z, wv.w};
    uint32_t oa[8], ob[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) decode8(wd[q], oa + 2 * q, ob + 2 * q);
    pa[2 * i] = make_uint4(oa[0], oa[1], oa[2], oa[3]);
    pa[2 * i + 1] = make_uint4(oa[4], oa[5], oa[6], oa[7]);
    pb[2 * i] = make_uint4(ob[0], ob[1], ob[2], ob[3]);
    pb[2 * i + 1] = make_uint4(ob[4], ob[5], ob[6], ob[7]);
}

// Workgroups of THREADS threads that a SideWork takes, and what workgroup `block` of them does (routing first: it takes
// longest).  Routing is part of it for two experts only.
template <int THREADS>
inline long side_blocks(const SideWork &w) {
    return (w.route.T + THREADS - 1) / THREADS + decode_blocks<THREADS>(w.decode) + (w.zero.n > 0 ? 1 : 0);
}
template <int THREADS>
__device__ __forceinline__ void side_block(const SideWork &w, long block) {
    const long route = (w.route.T + THREADS - 1) / THREADS, decode = decode_blocks<THREADS>(w.decode);
    if (block < route)
        route_scatter_block<THREADS, 2>(w.route, (int)block);
    else if (block < route + decode)
        decode_block<THREADS>(w.decode, block - route);
    else if (block == route + decode)
        zero_words(w.zero);
}

}  // namespace sa
