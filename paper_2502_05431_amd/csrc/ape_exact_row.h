// What the matrix-core kernels that are built on plain builtins and give every probability as the sum of two bf16 values (or in fp32)
// have in common beside the products: the score scale, and the loop on the vector ALUs that computes single rows again.
#pragma once

#include "ape_mfma.h"

#include <math.h>

#include <type_traits>

namespace ape {
namespace {

constexpr float kNone = -3.402823466e+38f;   // softmax reference of a row that has not seen a score yet: the lowest, so that every score can be one
constexpr float kFar = 0x1p27f;              // beyond this (either sign) the rounding of a reference alone is more than exp can take
constexpr float kSlack = 10.f;               // a reference moves only when exceeded by this (fp32 sums lose nothing by that)

// 1/(T sqrt d), rounded once.  Scores of |x| = 40 (T = 0.1) turn one rounding of the scale into 2.4e-6 of a probability, so
// fp32 carries its remainder along and keeps natural-log units (a factor log2 e inside would round once more);
// bf16 has log2 e inside and a single fused multiply per score.
template <typename T>
struct ScoreScale {
    static constexpr bool F32 = sizeof(T) == 4;
    float hi, lo;
    __device__ __forceinline__ ScoreScale(int d, float temperature) {
        const double x = (F32 ? 1.0 : 1.4426950408889634) / (sqrt((double)d) * (double)temperature);
        hi = (float)x; lo = (float)(x - (double)hi);
    }
    // exp of (difference of references)
    static __device__ __forceinline__ float exp_of(float x) { return __builtin_amdgcn_exp2f(F32 ? x * LOG2E : x); }
    __device__ __forceinline__ float prob(float s, float m) const {
        return exp_of(F32 ? fmaf(s, hi, fmaf(s, lo, -m)) : fmaf(s, hi, -m));
    }
    static __device__ __forceinline__ float lse(float m, float l) {
        const float x = __builtin_amdgcn_logf(l);            // log2
        return F32 ? fmaf(x, LN2, m) : (m + x) * LN2;
    }
};

// (the compiler is told that there are no NaNs: it is not shown where these bits come from)
__device__ __forceinline__ bool finite(float x) {
    uint32_t bits = __float_as_uint(x);
    asm("" : "+v"(bits));
    return (bits & 0x7fffffffu) < 0x7f800000u;
}

// Whether a row saw any token: a sum of probabilities that is not zero, be it not a number (the compiler is told that there are
// none, so the bits are asked).
__device__ __forceinline__ bool seen(float sum) {
    uint32_t bits = __float_as_uint(sum);
    asm("" : "+v"(bits));
    return bits != 0;
}

// A row's 4 consecutive output values, in the storage type.
__device__ __forceinline__ void store4(float* p, const float (&x)[4]) { *(f32x4*)p = f32x4{x[0], x[1], x[2], x[3]}; }
__device__ __forceinline__ void store4(__bf16* p, const float (&x)[4]) { *(u32x2*)p = u32x2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])}; }

__device__ __forceinline__ float lane_value(float x, int lane) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), lane)); }

// One row by a whole wavefront: scores with a token per lane, values with dims lane + 64 r per lane.  Natural-log units.
template <typename T>
struct ExactRow {
    static constexpr int E = 16 / (int)sizeof(T);
    float q[4], acc[4], m, l;
    int d;
    __device__ __forceinline__ ExactRow(const T* row, int d_) : m(-INFINITY), l(0.f), d(d_) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = (threadIdx.x & 63) + 64 * r;
            q[r] = c < d ? (float)row[c] : 0.f;
            acc[r] = 0.f;
        }
    }
    // n tokens, `stride` elements apart
    __device__ __forceinline__ void attend(const T* k, const T* v, long stride, int n, float scale) {
#pragma clang fp contract(off)
        const int lane = threadIdx.x & 63;
        for (int j0 = 0; j0 < n; j0 += 64) {
            const int cnt = min(64, n - j0);
            const T* kr = k + (long)(j0 + min(lane, cnt - 1)) * stride;
            float dot = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll 4
                for (int c = 64 * r; c < min(d, 64 * r + 64); c += E) {
                    T x[E];
                    *(u32x4*)x = *(const u32x4*)(kr + c);
#pragma unroll
                    for (int e = 0; e < E; ++e) dot = fmaf(lane_value(q[r], c - 64 * r + e), (float)x[e], dot);
                }
            const float s = lane < cnt ? dot * scale : -INFINITY;
            float m_new = s;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) m_new = fmaxf(m_new, __shfl_xor(m_new, o));
            m_new = fmaxf(m, m_new);
            if (m_new == -INFINITY) continue;                // masked tokens only
            // (the instructions, which keep a score that is no number: the library's functions may be compiled not to)
            const float p = lane < cnt ? __builtin_amdgcn_exp2f((s - m_new) * LOG2E) : 0.f, alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - m_new) * LOG2E);
            float sum = p;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
            m = m_new; l = l * alpha + sum;
            if (!finite(l)) return;                          // a seen score is no number: no more of it
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] *= alpha;
            int jj = 0;
            auto add_values = [&](auto few) {
                float x[few()][4];
#pragma unroll
                for (int u = 0; u < few(); ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[u][r] = lane + 64 * r < d ? (float)v[(long)(j0 + jj + u) * stride + lane + 64 * r] : 0.f;
#pragma unroll
                for (int u = 0; u < few(); ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[r] = fmaf(lane_value(p, jj + u), x[u][r], acc[r]);
                jj += few();
            };
            while (jj + 8 <= cnt) add_values(std::integral_constant<int, 8>());
            while (jj < cnt) add_values(std::integral_constant<int, 1>());
        }
    }
    __device__ __forceinline__ float lse() const { return seen(l) ? m + __builtin_amdgcn_logf(l) * LN2 : -INFINITY; }
    // as scale_contexts
    __device__ __forceinline__ void scale_contexts(float scale) {
        if (!seen(l)) return;
        const float inv = 1.f / l;
        m = scale * lse(); l = 1.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] *= inv;
    }
    // dims [c0, c1) of the normalised values
    template <typename OUT>
    __device__ __forceinline__ void store(OUT* o, int c0, int c1, float empty) const {
        const float inv = seen(l) ? 1.f / l : empty;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = (threadIdx.x & 63) + 64 * r;
            if (c >= c0 && c < min(c1, d)) o[c] = (OUT)(acc[r] * inv);
        }
    }
};

// `redo`: rows R0 + bit; dims [c0, c1) are this wavefront's.  The kernel's arguments are read again where they lie (through a pointer
// that the compiler cannot see through), so that nothing is kept for this over the streams.
template <typename Args>
__device__ __forceinline__ __attribute__((address_space(4))) const Args* kernarg_again() {
    auto a = kernarg<Args>();
    asm volatile("" : "+s"(a));
    return a;
}

// Query rows past context tokens [t0, t1) and, if `own`, then past the prefix and the own tokens; `whole`: this is the output (else
// the partial result whose rows begin at part0).
template <typename T, typename Args>
__device__ __forceinline__ void redo_query_rows(__attribute__((address_space(4))) const Args* a, int rq, int hk, long part0, int t0, int t1,
                                                bool own, bool whole, int R0, uint32_t redo, int c0, int c1) {
    const int d = a->head_dim, hq = a->n_q_heads, hkv = a->n_kv_heads, G = hq / hkv, q_len = a->q_len;
    const int n_chunks = a->req[rq].n_chunks;
    const int32_t* cu = a->req[rq].cu;
    const long stride = (long)hkv * d, head = (long)hk * d;
    const bool first_dims = c0 == 0 && (threadIdx.x & 63) == 0;
    for (; redo; redo &= redo - 1) {
        const int R = R0 + __builtin_ctz(redo), tok = R / G, h = hk * G + R % G;
        const long row = ((long)rq * q_len + tok) * hq + h, unit = (long)a->req_base * q_len * hq + row;
        ExactRow<T> x((const T*)a->q + row * d, d);
        const int last = own ? n_chunks + 2 : n_chunks;
        int t = t0;
        for (int c = t0 < t1 ? find_chunk(cu, n_chunks, t0) : n_chunks; c < last; ++c) {   // the contexts, the prefix, the own tokens
            const T *k, *v;
            int n;
            float scale = rsqrtf((float)d);
            if (c < n_chunks) {
                const int from = cu[c], to = min(cu[c + 1], t1);
                n = to - t;
                k = (const T*)a->req[rq].k_chunks[c] + (long)(t - from) * stride; v = (const T*)a->req[rq].v_chunks[c] + (long)(t - from) * stride;
                scale /= a->req[rq].temperature;
                t = max(t, to);
            } else if (c == n_chunks) {
                x.scale_contexts(a->req[rq].scale);
                n = a->req[rq].prefix_len;
                k = (const T*)a->req[rq].k_prefix; v = (const T*)a->req[rq].v_prefix;
            } else {
                n = a->req[rq].self_len - q_len + tok + 1;
                k = (const T*)a->req[rq].k_self; v = (const T*)a->req[rq].v_self;
            }
            x.attend(k + head, v + head, stride, n, scale);
        }
        if (whole) {
            x.store((T*)a->out + unit * d, c0, c1, INFINITY);
            if (a->lse_out && first_dims) a->lse_out[a->lse_head_major ? ((long)(a->req_base + rq) * hq + h) * q_len + tok : unit] = x.lse();
        } else {
            const long slot = part0 + (long)tok * hq + h;
            x.store(a->part_o + slot * d, c0, c1, 0.f);
            if (first_dims) a->part_lse[slot] = x.lse();
        }
    }
}

}  // namespace
}  // namespace ape
