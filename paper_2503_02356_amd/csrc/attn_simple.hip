// Plain scalar attention kernels for one chunk: fp32 arithmetic, fp32 or bf16 storage.
// One wavefront per query row (forward, dQ) or per key row (dK/dV).  They serve the cross-check flag and
// whatever the matrix kernels do not cover.
//
// Math (paper sections 2.1, 2.2, 4.2 give the masking and the state dependency; the formulas are
// the standard softmax-attention gradient):
//   query i of a segment sees keys j <= i + (Lk - Lq);  S = scale * q.k;  P = exp(S - LSE);
//   O = sum_j P v_j;  dV_j += sum_i P dO_i;  dS = P (dO_i.v_j - delta_i);
//   dQ_i = scale sum_j dS k_j;  dK_j += scale sum_i dS q_i.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "scalar_rows.h"

namespace cf {
namespace {

constexpr int kWaves = kScalarWaves;  // wavefronts per workgroup

// Largest g in [0, n) with cu[g] <= row  (cu non-decreasing, cu[0] = 0, zero-length segments skipped).
__device__ inline int find_segment(const int32_t *cu, int n, int row)
{
    int lo = 0, hi = n;  // invariant: cu[lo] <= row < cu[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cu[mid] <= row) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ inline SegmentRows segment_rows(const cf_attn_fwd_params &p, int g)
{
    const int q0 = p.cu_seqlens_q[g], k0 = p.cu_seqlens_k[g];
    return {q0, p.cu_seqlens_q[g + 1] - q0, k0, p.cu_seqlens_k[g + 1] - k0};
}
__device__ inline SegmentRows segment_of_query(const cf_attn_fwd_params &p, int row)
{
    return segment_rows(p, find_segment(p.cu_seqlens_q, p.n_segments, row));
}

template <typename T, int D>
__global__ __launch_bounds__(kWaves * 64) void simple_fwd_kernel(cf_attn_fwd_params p)
{
    __shared__ float sq[kWaves][D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * kWaves + wave;
    if (row >= p.n_tokens) return;  // whole wavefront leaves together; no barrier below
    const int h = blockIdx.y;
    const SegmentRows g = segment_of_query(p, row);
    const T *q = row_of<T>(p.q, row, p.q_stride_tok, h, p.q_stride_head);
    for (int t = 0; t < D / 64; ++t) sq[wave][lane + 64 * t] = ld(q + lane + 64 * t);
    __builtin_amdgcn_wave_barrier();
    scalar_fwd_row<T, D, 0>(p, g, row, h, [&](int x) { return sq[wave][x]; });
}

template <typename T, int D>
__global__ __launch_bounds__(kWaves * 64) void simple_dq_kernel(cf_attn_bwd_params b, const float *delta)
{
    const cf_attn_fwd_params &p = b.f;
    __shared__ float sq[kWaves][D], sdo[kWaves][D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * kWaves + wave;
    if (row >= p.n_tokens) return;
    const int h = blockIdx.y;
    const SegmentRows g = segment_of_query(p, row);
    const T *q = row_of<T>(p.q, row, p.q_stride_tok, h, p.q_stride_head);
    const T *d_o = row_of<T>(b.d_o, row, b.do_stride_tok, h, b.do_stride_head);
    for (int t = 0; t < D / 64; ++t) {
        sq[wave][lane + 64 * t] = ld(q + lane + 64 * t);
        sdo[wave][lane + 64 * t] = ld(d_o + lane + 64 * t);
    }
    __builtin_amdgcn_wave_barrier();
    scalar_dq_row<T, D, 0>(b, g, row, h, [&](int x) { return sq[wave][x]; }, [&](int x) { return sdo[wave][x]; },
                        delta[(int64_t)h * p.n_tokens + row]);
}

// One wavefront per (key row, key/value head): the only writer of that row of dK and dV.
template <typename T, int D>
__global__ __launch_bounds__(kWaves * 64) void simple_dkv_kernel(cf_attn_bwd_params b, const float *delta)
{
    const cf_attn_fwd_params &p = b.f;
    __shared__ float sk[kWaves][D], sv[kWaves][D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int krow = blockIdx.x * kWaves + wave;
    if (krow >= p.n_kv_tokens) return;
    const int kh = blockIdx.y, seg = find_segment(p.cu_seqlens_k, p.n_segments, krow);
    const SegmentRows g = segment_rows(p, seg);
    const T *k = row_of<T>(p.k, krow, p.kv_stride_tok, kh, p.kv_stride_head);
    const T *v = row_of<T>(p.v, krow, p.kv_stride_tok, kh, p.kv_stride_head);
    constexpr int DPL = D / 64;
    for (int t = 0; t < DPL; ++t) {
        sk[wave][lane + 64 * t] = ld(k + lane + 64 * t);
        sv[wave][lane + 64 * t] = ld(v + lane + 64 * t);
    }
    __builtin_amdgcn_wave_barrier();
    float dk[DPL], dv[DPL];
    scalar_dkv_row<T, D, 0>(b, g, krow, kh, [&](int x) { return sk[wave][x]; }, [&](int x) { return sv[wave][x]; },
                         [&](int row, int h) { return delta[(int64_t)h * p.n_tokens + row]; }, dk, dv);
    float *gk = b.d_k + (int64_t)krow * b.dkv_stride_tok + (int64_t)kh * b.dkv_stride_head;
    float *gv = b.d_v + (int64_t)krow * b.dkv_stride_tok + (int64_t)kh * b.dkv_stride_head;
    for (int t = 0; t < DPL; ++t) {
        gk[lane + 64 * t] += dk[t] * p.softmax_scale;
        gv[lane + 64 * t] += dv[t];
    }
}

// delta[h][t] = <dO_t, O_t>: 16 lanes per (token, head), 8 (or 4) consecutive d per lane and step.
template <typename T, int D>
__global__ __launch_bounds__(256) void delta_kernel(cf_attn_bwd_params b, float *delta)
{
    const cf_attn_fwd_params &p = b.f;
    const int64_t pair = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);   // (token, head) pair
    const int sub = threadIdx.x & 15;
    float s = 0.f;
    int64_t row = 0, h = 0;
    const bool live = pair < (int64_t)p.n_tokens * p.n_q_heads;
    if (live) {
        row = pair / p.n_q_heads;
        h = pair % p.n_q_heads;
        const T *o = (const T *)p.o + row * p.o_stride_tok + h * p.o_stride_head;
        const T *d_o = (const T *)b.d_o + row * b.do_stride_tok + h * b.do_stride_head;
        constexpr int V = 16 / sizeof(T);   // elements per 16-byte load
        for (int d0 = sub * V; d0 < D; d0 += 16 * V) {
            const uint4 a = *(const uint4 *)(o + d0), c = *(const uint4 *)(d_o + d0);
            const T *pa = (const T *)&a, *pc = (const T *)&c;
#pragma unroll
            for (int j = 0; j < V; ++j) s += ld(pa + j) * ld(pc + j);
        }
    }
    for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (live && sub == 0) delta[h * p.n_tokens + row] = s;
}

// O arrives rounded to the storage type, and for a row that sees only a few keys (large P, large |O|)
// that rounding would be the largest error of the whole backward pass (it lands in dK of the first keys of
// each sequence).  Rows that see at most 64 keys therefore get delta = sum_j P_tj <dO_t, v_j> instead,
// one key per lane, which needs no O at all.  One wavefront per (segment, one of its first 64 rows, head);
// runs after delta_kernel and overwrites its value for those rows (scalar backward path; the MFMA path
// does the same inside its dQ head blocks).
template <typename T, int D>
__global__ __launch_bounds__(kWaves * 64) void delta_head_rows_kernel(cf_attn_bwd_params b, float *delta)
{
    const cf_attn_fwd_params &p = b.f;
    __shared__ float sq[kWaves][D], sdo[kWaves][D];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int g = blockIdx.x / (64 / kWaves);
    const int i = (blockIdx.x % (64 / kWaves)) * kWaves + wave;        // row inside the segment, 0..63
    const int h = blockIdx.y;
    const int q0 = p.cu_seqlens_q[g], lq = p.cu_seqlens_q[g + 1] - q0;
    const int k0 = p.cu_seqlens_k[g], lk = p.cu_seqlens_k[g + 1] - k0;
    const int n_vis = lk - lq + i + 1;
    if (i >= lq || n_vis > 64) return;   // whole wavefront leaves together; only wave-level barriers below
    const int row = q0 + i;
    const int kh = h / (p.n_q_heads / p.n_kv_heads);
    const T *q = (const T *)p.q + (int64_t)row * p.q_stride_tok + (int64_t)h * p.q_stride_head;
    const T *d_o = (const T *)b.d_o + (int64_t)row * b.do_stride_tok + (int64_t)h * b.do_stride_head;
    for (int t = 0; t < D / 64; ++t) {
        sq[wave][lane + 64 * t] = ld(q + lane + 64 * t);
        sdo[wave][lane + 64 * t] = ld(d_o + lane + 64 * t);
    }
    __builtin_amdgcn_wave_barrier();
    float s = 0.f;
    if (lane < n_vis) {
        const T *kj = (const T *)p.k + (int64_t)(k0 + lane) * p.kv_stride_tok + (int64_t)kh * p.kv_stride_head;
        const T *vj = (const T *)p.v + (int64_t)(k0 + lane) * p.kv_stride_tok + (int64_t)kh * p.kv_stride_head;
        float sc = 0.f, dp = 0.f;
        for (int x = 0; x < D; ++x) {
            sc += sq[wave][x] * ld(kj + x);
            dp += sdo[wave][x] * ld(vj + x);
        }
        s = expf(sc * p.softmax_scale - p.lse[(int64_t)h * p.n_tokens + row]) * dp;
    }
    s = wave_sum(s);
    if (lane == 0) delta[(int64_t)h * p.n_tokens + row] = s;
}

template <typename T, int D>
hipError_t run_fwd(const cf_attn_fwd_params &p, hipStream_t s)
{
    dim3 grid((p.n_tokens + kWaves - 1) / kWaves, p.n_q_heads);
    const ProfileHook hook = take_profile_hook();
    if (hook.start) (void)hipEventRecord(hook.start, s);
    simple_fwd_kernel<T, D><<<grid, kWaves * 64, 0, s>>>(p);
    const hipError_t e = hipGetLastError();
    if (hook.stop) (void)hipEventRecord(hook.stop, s);
    return e;
}

template <typename T, int D>
hipError_t run_bwd(const cf_attn_bwd_params &b, const BwdWorkspace &ws, hipStream_t s)
{
    const cf_attn_fwd_params &p = b.f;
    // exact delta for rows that see at most 64 keys (overwrites delta_kernel's value for them)
    dim3 gh(p.n_segments * (64 / kWaves), p.n_q_heads);
    delta_head_rows_kernel<T, D><<<gh, kWaves * 64, 0, s>>>(b, ws.delta);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    dim3 gq((p.n_tokens + kWaves - 1) / kWaves, p.n_q_heads);
    const ProfileHook hook = take_profile_hook();
    if (hook.start) (void)hipEventRecord(hook.start, s);
    simple_dq_kernel<T, D><<<gq, kWaves * 64, 0, s>>>(b, ws.delta);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        dim3 gk((p.n_kv_tokens + kWaves - 1) / kWaves, p.n_kv_heads);
        simple_dkv_kernel<T, D><<<gk, kWaves * 64, 0, s>>>(b, ws.delta);
        e = hipGetLastError();
    }
    if (hook.stop) (void)hipEventRecord(hook.stop, s);
    return e;
}

template <typename T, int D>
hipError_t run_delta(const cf_attn_bwd_params &b, const BwdWorkspace &ws, hipStream_t s)
{
    const int64_t pairs = (int64_t)b.f.n_tokens * b.f.n_q_heads;
    delta_kernel<T, D><<<dim3((unsigned)((pairs + 15) / 16)), 256, 0, s>>>(b, ws.delta);
    return hipGetLastError();
}

}  // namespace

#define CF_DISPATCH(fn, dtype, D, ...)                                              \
    do {                                                                            \
        if ((dtype) == CF_FP32 && (D) == 64) return fn<float, 64>(__VA_ARGS__);     \
        if ((dtype) == CF_FP32 && (D) == 128) return fn<float, 128>(__VA_ARGS__);   \
        if ((dtype) == CF_BF16 && (D) == 64) return fn<unsigned short, 64>(__VA_ARGS__);   \
        if ((dtype) == CF_BF16 && (D) == 128) return fn<unsigned short, 128>(__VA_ARGS__); \
        return hipErrorInvalidValue;                                                \
    } while (0)

hipError_t launch_simple_fwd(const cf_attn_fwd_params &p, hipStream_t s)
{
    CF_DISPATCH(run_fwd, p.dtype, p.head_dim, p, s);
}
hipError_t launch_simple_bwd(const cf_attn_bwd_params &b, const BwdWorkspace &ws, hipStream_t s)
{
    CF_DISPATCH(run_bwd, b.f.dtype, b.f.head_dim, b, ws, s);
}
hipError_t launch_delta(const cf_attn_bwd_params &b, const BwdWorkspace &ws, hipStream_t s)
{
    CF_DISPATCH(run_delta, b.f.dtype, b.f.head_dim, b, ws, s);
}

}  // namespace cf
