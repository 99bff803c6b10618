// Attention of single rows by one wavefront, in fp32 arithmetic and pair by pair: a pair that the causal mask hides is never
// read.  The scalar kernels are made of these; the matrix kernels that stand in for them take a row from here when its result
// is not finite: they multiply whole blocks, hidden pairs by zero, and zero times an infinity or a NaN of a later row would
// reach rows that do not see it.
//   B  the parameters of a backward call: cf_attn_bwd_params or what a kernel takes of it (BwdArgs)
//   row operands are passed as functions of the element index (LDS copies, or the global row itself)
//   UNROLL  of the loops over the elements of a row: small in the matrix kernels, whose registers are not to be spilled for it
#pragma once
#include <hip/hip_runtime.h>

#include "chunkflow.h"

namespace cf {

__device__ inline float ld(const float *p) { return *p; }
__device__ inline float ld(const unsigned short *p) { return __uint_as_float(((unsigned)*p) << 16); }
__device__ inline void st(float *p, float x) { *p = x; }
__device__ inline void st(unsigned short *p, float x)
{  // round to nearest even bf16
    unsigned u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    *p = (unsigned short)(u >> 16);
}

__device__ inline float wave_max(float x)
{
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}
__device__ inline float wave_sum(float x)
{
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// UNROLL 0: as the compiler likes.
template <int D, int UNROLL, typename F>
__device__ inline void for_elements(F f)
{
    if constexpr (UNROLL == 0) {
        for (int x = 0; x < D; ++x) f(x);
    } else {
#pragma unroll UNROLL
        for (int x = 0; x < D; ++x) f(x);
    }
}

// Rows of a segment in the call's tensors: queries [q0, q0 + lq), keys [k0, k0 + lk).
struct SegmentRows {
    int q0, lq, k0, lk;
};
template <typename T>
__device__ inline const T *row_of(const void *base, int row, int64_t stride_tok, int head, int64_t stride_head)
{
    return (const T *)base + (int64_t)row * stride_tok + (int64_t)head * stride_head;
}

// O and LSE of query row `row` of head h.
template <typename T, int D, int UNROLL, typename Q>
__device__ inline void scalar_fwd_row(const cf_attn_fwd_params &p, const SegmentRows &g, int row, int h, Q q)
{
    const int lane = threadIdx.x & 63, kh = h / (p.n_q_heads / p.n_kv_heads);
    const int n_vis = g.lk - g.lq + (row - g.q0) + 1;
    const T *kb = (const T *)p.k + (int64_t)kh * p.kv_stride_head;
    const T *vb = (const T *)p.v + (int64_t)kh * p.kv_stride_head;
    constexpr int DPL = D / 64;
    float m = -INFINITY, z = 0.f, acc[DPL];
    for (int t = 0; t < DPL; ++t) acc[t] = 0.f;
    for (int j0 = 0; j0 < n_vis; j0 += 64) {
        const int j = j0 + lane;
        float s = -INFINITY;
        if (j < n_vis) {
            const T *kj = kb + (int64_t)(g.k0 + j) * p.kv_stride_tok;
            float d = 0.f;
            for_elements<D, UNROLL>([&](int x) { d += q(x) * ld(kj + x); });
            s = d * p.softmax_scale;
        }
        const float m_new = fmaxf(m, wave_max(s));
        const float pr = (j < n_vis) ? expf(s - m_new) : 0.f;
        const float corr = expf(m - m_new);  // m = -inf on the first block gives 0
        z = z * corr + wave_sum(pr);
        for (int t = 0; t < DPL; ++t) acc[t] *= corr;
        const int cnt = min(64, n_vis - j0);
        for (int jj = 0; jj < cnt; ++jj) {
            const float pj = __shfl(pr, jj);
            const T *vj = vb + (int64_t)(g.k0 + j0 + jj) * p.kv_stride_tok;
            for (int t = 0; t < DPL; ++t) acc[t] += pj * ld(vj + lane + 64 * t);
        }
        m = m_new;
    }
    T *o = (T *)p.o + (int64_t)row * p.o_stride_tok + (int64_t)h * p.o_stride_head;
    const float inv = 1.f / z;
    for (int t = 0; t < DPL; ++t) st(o + lane + 64 * t, acc[t] * inv);
    if (lane == 0) p.lse[(int64_t)h * p.n_tokens + row] = m + logf(z);
}

// dQ of query row `row` of head h.
template <typename T, int D, int UNROLL, typename B, typename Q, typename DO>
__device__ inline void scalar_dq_row(const B &b, const SegmentRows &g, int row, int h, Q q, DO d_o, float delta)
{
    const auto &p = b.f;
    const int lane = threadIdx.x & 63, kh = h / (p.n_q_heads / p.n_kv_heads);
    const int n_vis = g.lk - g.lq + (row - g.q0) + 1;
    const T *kb = (const T *)p.k + (int64_t)kh * p.kv_stride_head;
    const T *vb = (const T *)p.v + (int64_t)kh * p.kv_stride_head;
    constexpr int DPL = D / 64;
    const float lse = p.lse[(int64_t)h * p.n_tokens + row];
    float acc[DPL];
    for (int t = 0; t < DPL; ++t) acc[t] = 0.f;
    for (int j0 = 0; j0 < n_vis; j0 += 64) {
        const int j = j0 + lane;
        float ds = 0.f;
        if (j < n_vis) {
            const T *kj = kb + (int64_t)(g.k0 + j) * p.kv_stride_tok;
            const T *vj = vb + (int64_t)(g.k0 + j) * p.kv_stride_tok;
            float s = 0.f, dp = 0.f;
            for_elements<D, UNROLL>([&](int x) {
                s += q(x) * ld(kj + x);
                dp += d_o(x) * ld(vj + x);
            });
            ds = expf(s * p.softmax_scale - lse) * (dp - delta);
        }
        const int cnt = min(64, n_vis - j0);
        for (int jj = 0; jj < cnt; ++jj) {
            const float dj = __shfl(ds, jj);
            const T *kj = kb + (int64_t)(g.k0 + j0 + jj) * p.kv_stride_tok;
            for (int t = 0; t < DPL; ++t) acc[t] += dj * ld(kj + lane + 64 * t);
        }
    }
    T *dq = (T *)b.d_q + (int64_t)row * b.dq_stride_tok + (int64_t)h * b.dq_stride_head;
    for (int t = 0; t < DPL; ++t) st(dq + lane + 64 * t, acc[t] * p.softmax_scale);
}

// What all query heads of key/value head kh add to dK and dV of key row `krow` (element lane + 64 t; dK without the scale).
// delta(row, h): of a query row.
template <typename T, int D, int UNROLL, typename B, typename K, typename V, typename Delta>
__device__ inline void scalar_dkv_row(const B &b, const SegmentRows &g, int krow, int kh, K k, V v, Delta delta,
                                      float (&dk)[D / 64], float (&dv)[D / 64])
{
    const auto &p = b.f;
    const int lane = threadIdx.x & 63, G = p.n_q_heads / p.n_kv_heads;
    const int j = krow - g.k0, prefix = g.lk - g.lq;
    const int i_first = j > prefix ? j - prefix : 0;  // first query row that sees this key
    constexpr int DPL = D / 64;
    for (int t = 0; t < DPL; ++t) dk[t] = dv[t] = 0.f;
    for (int h = kh * G; h < (kh + 1) * G; ++h) {
        const T *qb = (const T *)p.q + (int64_t)h * p.q_stride_head;
        const T *dob = (const T *)b.d_o + (int64_t)h * b.do_stride_head;
        for (int i0 = i_first; i0 < g.lq; i0 += 64) {
            const int i = i0 + lane;
            float pr = 0.f, ds = 0.f;
            if (i < g.lq) {
                const T *qi = qb + (int64_t)(g.q0 + i) * p.q_stride_tok;
                const T *doi = dob + (int64_t)(g.q0 + i) * b.do_stride_tok;
                float s = 0.f, dp = 0.f;
                for_elements<D, UNROLL>([&](int x) {
                    s += ld(qi + x) * k(x);
                    dp += ld(doi + x) * v(x);
                });
                pr = expf(s * p.softmax_scale - p.lse[(int64_t)h * p.n_tokens + g.q0 + i]);
                ds = pr * (dp - delta(g.q0 + i, h));
            }
            const int cnt = min(64, g.lq - i0);
            for (int ii = 0; ii < cnt; ++ii) {
                const float pi = __shfl(pr, ii), di = __shfl(ds, ii);
                const T *qi = qb + (int64_t)(g.q0 + i0 + ii) * p.q_stride_tok;
                const T *doi = dob + (int64_t)(g.q0 + i0 + ii) * b.do_stride_tok;
                for (int t = 0; t < DPL; ++t) {
                    dv[t] += pi * ld(doi + lane + 64 * t);
                    dk[t] += di * ld(qi + lane + 64 * t);
                }
            }
        }
    }
}

// delta of a query row, formed by each lane for itself: <dO, O>, and for rows that see at most 64 keys sum_j P_j <dO, v_j>.
template <typename T, int D, typename B>
__device__ inline float scalar_delta(const B &b, const SegmentRows &g, int row, int h)
{
    const auto &p = b.f;
    const int n_vis = g.lk - g.lq + (row - g.q0) + 1, kh = h / (p.n_q_heads / p.n_kv_heads);
    const T *d_o = row_of<T>(b.d_o, row, b.do_stride_tok, h, b.do_stride_head);
    float sum = 0.f;
    if (n_vis > 64) {
        const T *o = row_of<T>(p.o, row, p.o_stride_tok, h, p.o_stride_head);
#pragma unroll 4
        for (int x = 0; x < D; ++x) sum += ld(o + x) * ld(d_o + x);
        return sum;
    }
    const T *q = row_of<T>(p.q, row, p.q_stride_tok, h, p.q_stride_head);
    const float lse = p.lse[(int64_t)h * p.n_tokens + row];
    for (int j = 0; j < n_vis; ++j) {
        const T *k = row_of<T>(p.k, g.k0 + j, p.kv_stride_tok, kh, p.kv_stride_head);
        const T *v = row_of<T>(p.v, g.k0 + j, p.kv_stride_tok, kh, p.kv_stride_head);
        float s = 0.f, dp = 0.f;
#pragma unroll 4
        for (int x = 0; x < D; ++x) {
            s += ld(q + x) * ld(k + x);
            dp += ld(d_o + x) * ld(v + x);
        }
        sum += expf(s * p.softmax_scale - lse) * dp;
    }
    return sum;
}

__device__ inline bool finite(float x) { return fabsf(x) < INFINITY; }

}  // namespace cf
