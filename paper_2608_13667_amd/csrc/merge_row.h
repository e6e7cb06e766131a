// Log-sum-exp merge of one output row from its partial results: the second stage of fork-aware
// decode attention (the merge kernel runs one block per output row).
//
// A part p of row (s, h) holds the row's attention over a disjoint set of its keys: the
// normalised output o_p and lse_p = ln(sum of exp(score)) over that set.  Their union is
//   M = max_p lse_p,  w_p = exp(lse_p - M),  o = sum_p w_p o_p / sum_p w_p,  lse = M + ln sum_p w_p.
// A part with lse = -inf holds no keys and has weight 0; if every part is empty the row has no
// keys at all and gets o = 0, lse = -inf.  A NaN part propagates.  In a fused step the token
// being appended is one more part, o = v_new, lse = scale * q . k_new, read from k_new / v_new
// (it is stored into the cache after every block of the step has read the lengths).
#pragma once

#include <type_traits>

#include "internal.h"

namespace fka {

typedef float merge_f32x4 __attribute__((ext_vector_type(4)));

struct RowMerge {
    const float *part_o;    // part j of the row at part_o[(p_first + j * p_step) * HD]
    const float *part_lse;  // ... and part_lse[p_first + j * p_step]
    uint32_t p_first, p_step;  // byte offsets of the parts are below 2^31
    int n;                  // parts
    // fused step (the token appended this step joins as one more part when its sequence has room)
    const int32_t *len;     // the sequence's length
    int max_len;
    const uint16_t *q_row;  // bf16 [HD]
    const uint16_t *k_row;  // bf16 [HD] k_new of the row's (sequence, KV head)
    const uint16_t *v_row;  // bf16 [HD]
    float scale;            // softmax scale (natural-log units)
    float *out_row;         // fp32 [HD]
    float *out_lse;         // fp32, nullable
};

// A reduction over the wave in vector-ALU steps (a shuffle is an LDS round trip): the halves, the
// 16-lane rows, then within a row.
template <class Op>
__device__ inline float fold32(float x, Op op)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return op(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
template <class Op>
__device__ inline float fold16(float x, Op op)
{
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
template <class Op>
__device__ inline float wave_reduce(float x, Op op)
{
    x = fold16(fold32(x, op), op);
    auto ror = [](float v, auto n) {  // the row rotated by n lanes (DPP row_ror)
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + decltype(n)::value, 0xf, 0xf, false));
    };
    x = op(x, ror(x, std::integral_constant<int, 8>{}));
    x = op(x, ror(x, std::integral_constant<int, 4>{}));
    x = op(x, ror(x, std::integral_constant<int, 2>{}));
    x = op(x, ror(x, std::integral_constant<int, 1>{}));
    return x;
}

// LDS the routine uses: each wave's sums and the maximum they are relative to.
template <int HD>
struct MergeLds {
    static constexpr int CH = HD / 4;    // float4 chunks per row
    static constexpr int SL = 256 / CH;  // part slices: slice k takes parts k, k + SL, ...
    merge_f32x4 acc[4][CH];
    float m[4], w[4];
};

// Merges row m with a block of 256 threads (every thread must call it), U parts of a slice requested
// at a time.
//
// What bounds a merge of few rows is latency: its bytes are in L2 or the Infinity Cache, and each load
// that waits for another costs 0.7-1 us.  So everything is requested before anything is waited for,
// branch-free (a part past the end reads at an offset past the buffer's range, which returns 0): the
// appended token's inputs and the thread's parts with their lse.  A wave's slices are joined in registers
// (one maximum for the wave, so their sums add up as they are), the waves through LDS at one barrier.
// (Every wave reading all the lse values lane-wise instead, to know the row's maximum in front, is
// as fast for few rows and slower for many: it doubles the requests to L2.)
template <int HD, bool STEP, int U>
__device__ inline void merge_row_by(const RowMerge &m, MergeLds<HD> &lds)
{
    constexpr int CH = MergeLds<HD>::CH, SL = MergeLds<HD>::SL;
    constexpr float kLog2eM = 1.442695040888963407f;
    constexpr uint32_t kPast = 0x80000000u;  // past the range of the descriptors below
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = tid % CH, slice = tid / CH;
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((void *)m.part_o, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc((void *)m.part_lse, 0, 0x7fffffff, 0x00020000);
    auto past = [&](int j) { return (uint32_t)(m.n - 1 - j) & kPast; };  // for a part past the end
    auto part = [&](int j) { return m.p_first + (uint32_t)j * m.p_step; };
    auto lse_at = [&](int j) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rl, (part(j) * 4) | past(j), 0, 0)); };
    auto o_at = [&](int j) {
        return __builtin_bit_cast(merge_f32x4,
                                  __builtin_amdgcn_raw_buffer_load_b128(ro, ((part(j) * HD + 4 * chunk) * 4) | past(j), 0, 0));
    };
    auto max_of = [](float a, float b) { return fmaxf(a, b); };
    auto sum_of = [](float a, float b) { return a + b; };
    // over the wave's slices: lanes of one chunk
    auto slices = [&](float x, auto op) {
        x = fold32(x, op);
        if constexpr (HD == 64) x = fold16(x, op);
        return x;
    };

    [[maybe_unused]] int len = 0;
    [[maybe_unused]] uint32_t q2 = 0, k2 = 0;
    [[maybe_unused]] uint2 new_v = {0, 0};
    if constexpr (STEP) {
        if (wave == 0) {  // it writes the row
            // a vector load: a scalar one would be waited for where it is made uniform
            int zero = 0;
            asm("" : "+v"(zero));
            len = m.len[zero];
            if constexpr (HD == 128) {
                q2 = reinterpret_cast<const uint32_t *>(m.q_row)[lane];
                k2 = reinterpret_cast<const uint32_t *>(m.k_row)[lane];
            } else {
                q2 = (uint32_t)m.q_row[lane] << 16;
                k2 = (uint32_t)m.k_row[lane] << 16;
            }
            new_v = *reinterpret_cast<const uint2 *>(m.v_row + 4 * chunk);
        }
    }
    float l[U];
    merge_f32x4 o[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        l[u] = lse_at(slice + u * SL);
        o[u] = o_at(slice + u * SL);
    }

    // this thread's slice, relative to the wave's maximum so far
    float M = -INFINITY, W = 0.f;
    merge_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0;;) {
        float mn = M;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + slice + u * SL >= m.n) l[u] = -INFINITY;
            mn = fmaxf(mn, l[u]);
        }
        mn = slices(mn, max_of);
        const float mu = (mn == -INFINITY) ? 0.f : mn;
        if (j0 > 0) {
            const float sc = (M == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f((M - mu) * kLog2eM);
            W *= sc;
            acc *= sc;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float e = __builtin_amdgcn_exp2f((l[u] - mu) * kLog2eM);  // 0 for an empty part
            W += e;
            acc += e * (l[u] == -INFINITY ? merge_f32x4{0.f, 0.f, 0.f, 0.f} : o[u]);  // (nothing wrote its o)
        }
        M = mn;
        j0 += U * SL;
        if (j0 >= m.n) break;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            l[u] = lse_at(j0 + slice + u * SL);
            o[u] = o_at(j0 + slice + u * SL);
        }
    }
    W = slices(W, sum_of);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = slices(acc[i], sum_of);
    if (wave != 0 && lane < CH) {
        lds.acc[wave][lane] = acc;
        if (lane == 0) {
            lds.m[wave] = M;
            lds.w[wave] = W;
        }
    }
    [[maybe_unused]] float s_new = -INFINITY;
    if constexpr (STEP) {
        if (wave == 0) {
            float dot = __uint_as_float(q2 & 0xffff0000u) * __uint_as_float(k2 & 0xffff0000u);
            if constexpr (HD == 128) dot += __uint_as_float(q2 << 16) * __uint_as_float(k2 << 16);
            dot = wave_reduce(dot, sum_of);
            if (len < m.max_len) s_new = dot * m.scale;
        }
    }
    __syncthreads();
    if (tid >= CH) return;
    float mw[4] = {M, lds.m[1], lds.m[2], lds.m[3]}, Mr = fmaxf(s_new, M);
#pragma unroll
    for (int w = 1; w < 4; ++w) Mr = fmaxf(Mr, mw[w]);
    const float Mu = (Mr == -INFINITY) ? 0.f : Mr;
    merge_f32x4 t = {0.f, 0.f, 0.f, 0.f};
    float Wr = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        // (a wave without a maximum has no keys, W = 0, or a NaN part)
        const float e = (mw[w] == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f((mw[w] - Mu) * kLog2eM);
        t += e * (w == 0 ? acc : lds.acc[w][tid]);
        Wr += e * (w == 0 ? W : lds.w[w]);
    }
    if constexpr (STEP) {
        const float e = __builtin_amdgcn_exp2f((s_new - Mu) * kLog2eM);  // 0 without room
        Wr += e;
        if (s_new != -INFINITY)
            t += e * merge_f32x4{__uint_as_float(new_v.x << 16), __uint_as_float(new_v.x & 0xffff0000u),
                                 __uint_as_float(new_v.y << 16), __uint_as_float(new_v.y & 0xffff0000u)};
    }
    const merge_f32x4 r = (Wr == 0.f) ? merge_f32x4{0.f, 0.f, 0.f, 0.f} : t * __builtin_amdgcn_rcpf(Wr);
    *reinterpret_cast<merge_f32x4 *>(m.out_row + 4 * tid) = r;
    if (m.out_lse && tid == 0) *m.out_lse = (Wr == 0.f) ? -INFINITY : Mu + logf(Wr);
}

// As many loads in flight as the parts ask for (a slice of one part each; four; eight at a time).
template <int HD, bool STEP>
__device__ inline void merge_row(const RowMerge &m, MergeLds<HD> &lds)
{
    constexpr int SL = MergeLds<HD>::SL;
    if (m.n <= SL)
        merge_row_by<HD, STEP, 1>(m, lds);
    else if (m.n <= 4 * SL)
        merge_row_by<HD, STEP, 4>(m, lds);
    else
        merge_row_by<HD, STEP, 8>(m, lds);
}

}  // namespace fka
