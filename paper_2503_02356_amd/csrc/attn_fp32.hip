// fp32 attention for one chunk on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32 operands and sums, 64 FLOP
// per clock and SIMD, 32 clocks each), head_dim 64 and 128, any softmax scale.
//
// What bounds it: large calls the fp32 matrix rate (157 TFLOP/s) and how evenly the units below fill 256 compute units;
// small ones the serial chain of a wavefront (a 16 x 16 block of pairs is D / 4 dependent MFMAs per product) and the
// latency of its loads.  The unit of work is therefore small and split as far as it goes: ONE workgroup of 16 wavefronts
// owns 16 query rows of a head (forward, dQ) or 16 key rows of a key/value head (dK/dV), its wavefronts take every 16th
// block of the other side, and their partial results meet in LDS at the end in a fixed order: no atomics, every result
// has one writer and is bitwise reproducible.  (32-row units on 32x32x2 MFMAs would leave half the chip idle on a
// 700-row slice of 6 heads that is launched on its own: 132 workgroups.)
// Operands go straight from global memory into registers: a wavefront's blocks are its own, so LDS tiles would not be
// shared.  What the 16 wavefronts share, the owned rows, is kept in LDS in operand order.  The backward takes a block's rows in
// two orders, as rows and as columns: they are fetched once, and each wavefront turns them around in a piece of LDS of its own, where
// its result goes in the end (a second fetch made 40 instead of 24 KB per block of dK/dV at D = 128, 40 bytes per clock and compute
// unit at the full matrix rate: the two steps below 51.4 -> 45.6 us and 889 -> 790 us, the same bits).
//
// Everything is computed with the owned row on the lane axis, as in the bf16 kernels:
//   forward  S^T = K Q^T              O^T  += V^T P^T           lane % 16 = query
//   dQ       S^T, dP^T = V dO^T       dQ^T += K^T dS^T          lane % 16 = query
//   dK/dV    S = Q K^T, dP = dO V^T   dV^T += dO^T P, dK^T += Q^T dS   lane % 16 = key
// so that P and dS feed the second product from the registers the first one left them in: register i of a 16 x 16
// result holds row 4 * quarter + i (quarter = lane / 16), which is exactly the contraction index that a lane of that
// quarter supplies in step i.  The order of the contraction over d, and of the columns of a result, is free: both are
// chosen so that every global access is a float4.
//
// The backward is ONE launch: every workgroup forms delta = <dO, O> of the rows it meets itself (128 FMAs a row next to
// the MFMAs of four products), so that neither half waits for the other.
// Errors against fp64 are no larger than the scalar kernels' (step of 1 head, D = 64, 1286 tokens, relative: dQ 3.2e-7, dK 3.5e-7,
// dV 2.6e-7, O 1.8e-7; scalar 3.3e-7, 3.8e-7, 3.2e-7, 2.0e-7).
//
// Measured, forward + backward of a whole step, calls sharing launches: 6 chunks, 1286 tokens, 1 head, D = 64: 764 us -> 46 us;
// 6 / 2 heads, D = 128, 4799 tokens in 6 chunks: 13.7 ms -> 0.76 ms (before: one wavefront per row, scalar loads;
// attn_simple.hip).
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "mfma_common.h"
#include "scalar_rows.h"

namespace cf {
namespace {

constexpr int NW = 16;           // wavefronts per workgroup
constexpr int RB = 16;           // rows per block
constexpr int kExactDeltaKeys = 64;      // rows that see at most so many keys: dQ takes delta from P and dP (as the scalar kernels do)
constexpr float kNoRow = 1e30f;  // LSE of a row past the end: P = 0 (finite, so that probability() takes no difference of infinities)
constexpr float kLog2e = 1.44269504088896340736f;
constexpr float kLn2 = 0.69314718055994530942f;

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int D>
struct Shape {
    static constexpr int J = D / 16;         // float4 pieces of a row that a lane holds (quarter rows)
    static constexpr int NC = D / 64;        // 64-wide column groups of a result
    static constexpr int OS = D + 4;         // row stride of a partial result in LDS (spreads float4 rows over the banks)
    static constexpr int PART = RB * OS;     // floats of one wavefront's partial result
    static constexpr int OPERAND = RB * D * 4;   // bytes of 16 staged rows
    static constexpr int OPERANDS = 2 * OPERAND + RB * 4;    // what the backward stages: two operands, delta
    static constexpr bool BOTH_MEET = D == 64;   // LDS holds the partial results of dK and dV at once
};
template <int D>
using Acc = f32x4[D / 16];                   // [4 * c + e], register i: column 64 c + 4 * (4 * quarter + i) + e

// The lane, as a value that the compiler does not know to be the same for every item: what follows from it is formed where it is used.
template <int USE>
__device__ __forceinline__ int lane_again(int lane, int item)
{
    int x;
    asm("; lane %c3" : "=v"(x) : "0"(lane), "s"(item), "n"(USE));
    return x;
}

// Combines over the 16 lanes of a quarter (rotations inside a row of 16 lanes).
template <int N>
__device__ __forceinline__ float add_rotated(float x)
{
    return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float sum_over_16_lanes(float x) { return add_rotated<1>(add_rotated<2>(add_rotated<4>(add_rotated<8>(x)))); }

// This lane's quarter of a row: floats 16 j + 4 * quarter + 0..3.
template <int D>
__device__ __forceinline__ void load_row(const float *row, int quarter, f32x4 (&f)[D / 16])
{
#pragma unroll
    for (int j = 0; j < D / 16; ++j) f[j] = *(const f32x4 *)(row + 16 * j + 4 * quarter);
}
// The 16 owned rows into LDS, in operand order: piece c (floats 4 c .. 4 c + 3) of row r at [c * 16 + r].
template <int D, bool ANEW = false>
__device__ __forceinline__ void stage_rows(const float *base, int64_t stride, int row0, int last_row, f32x4 *dst)
{
    for (int t = ANEW ? wave_id() * 64 + fresh_lane() : threadIdx.x; t < RB * D / 4; t += NW * 64) {
        const int r = t / (D / 4), c = t % (D / 4);
        dst[c * RB + r] = *(const f32x4 *)(base + (int64_t)min(row0 + r, last_row) * stride + c * 4);
    }
}
// rows (A operand, from registers) x owned rows (B operand, from LDS), contraction over d.
template <int D>
__device__ __forceinline__ f32x4 row_product(const f32x4 (&a)[D / 16], const f32x4 *b, int lane)
{
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < D / 16; ++j) {
        const f32x4 bj = b[j * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = mfma_f32(a[j][e], bj[e], acc);
    }
    return acc;
}
// Column operands of a 16-row block: whole rows per 16 lanes, step i of the contraction over the rows takes rows
// 4 * quarter + i, which is where register i of the other operand stands; lane % 16 = m holds columns 64 c + 4 m + e.
// Rows past last_row (relative to the block's first row, `block`) re-read last_row; the other operand is 0 there.
// (A scalar base that is known to be global memory and a 32-bit lane offset: a flat load would also wait for LDS.)
template <int D>
__device__ __forceinline__ void load_columns(const float *block, unsigned row_bytes, int last_row, int lane, f32x4 (&x)[4][D / 64])
{
    const int quarter = lane >> 4, m = lane & 15;
    const CF_GLOBAL char *base = (const CF_GLOBAL char *)uniform(block);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < D / 64; ++c)
            x[i][c] = *(const CF_GLOBAL f32x4 *)(base + ((unsigned)min(4 * quarter + i, last_row) * row_bytes + 16 * m + 256 * c));
}
// The same columns of rows that this wavefront already holds (load_row), turned around through its own piece of LDS.  In two
// parts: the rows may leave their registers in between.
__device__ __forceinline__ void lds_turn() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"), __builtin_amdgcn_wave_barrier(); }
template <int D>
__device__ __forceinline__ void put_rows(const f32x4 (&f)[D / 16], float *piece, int lane)
{
    lds_turn();                                      // (what stood there has been read)
#pragma unroll
    for (int j = 0; j < D / 16; ++j) *(f32x4 *)(piece + (lane & 15) * Shape<D>::OS + 16 * j + 4 * (lane >> 4)) = f[j];
    lds_turn();
}
// acc^T += X^T w
template <int D>
__device__ __forceinline__ void add_column_product(const f32x4 (&x)[4][D / 64], const f32x4 &w, Acc<D> &acc)
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < D / 64; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * c + e] = mfma_f32(x[i][c][e], w[i], acc[4 * c + e]);
}
// acc^T += X^T w, X the rows that stand in this wavefront's piece of LDS
template <int D>
__device__ __forceinline__ void add_column_product(const float *piece, int lane, const f32x4 &w, Acc<D> &acc)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (D != 64) __builtin_amdgcn_sched_barrier(0);  // (all of X at once: 34 registers spilled)
        f32x4 x[D / 64];
#pragma unroll
        for (int c = 0; c < D / 64; ++c) x[c] = *(const f32x4 *)(piece + (4 * (lane >> 4) + i) * Shape<D>::OS + 4 * (lane & 15) + 64 * c);
#pragma unroll
        for (int c = 0; c < D / 64; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * c + e] = mfma_f32(x[c][e], w[i], acc[4 * c + e]);
    }
}
// A wavefront's transposed result (lane % 16 = owned row) into its part of the LDS scratch.
template <int D>
__device__ __forceinline__ void write_part(const Acc<D> &acc, float *part, int lane)
{
    const int quarter = lane >> 4, r = lane & 15;
#pragma unroll
    for (int c = 0; c < D / 64; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *(f32x4 *)(part + r * Shape<D>::OS + 64 * c + 16 * quarter + 4 * i) =
                f32x4{acc[4 * c][i], acc[4 * c + 1][i], acc[4 * c + 2][i], acc[4 * c + 3][i]};
}
template <int D>
__device__ __forceinline__ f32x4 sum_parts(const float *parts, int n, int row, int c)
{
    f32x4 s = *(const f32x4 *)(parts + row * Shape<D>::OS + c * 4);
    for (int w = 1; w < n; ++w) s += *(const f32x4 *)(parts + w * Shape<D>::PART + row * Shape<D>::OS + c * 4);
    return s;
}

// The last step of every kernel gives D / 4 consecutive lanes of a wavefront one row: visit(first lane of the row), by the whole
// wavefront, for every row that one of `lanes` has a part of.  (Rows whose result is not finite: see scalar_rows.h.)
template <int D>
__device__ __forceinline__ unsigned long long lanes_of_row(int lane) { return ((1ull << (D / 4)) - 1) << (lane / (D / 4) * (D / 4)); }
template <int D, typename Visit>
__device__ __forceinline__ void for_rows_of(unsigned long long lanes, Visit visit)
{
    static_assert(RB * (D / 4) <= NW * 64, "one step");
    while (lanes != 0) {
        const int first = __ffsll((long long)lanes) - 1;
        lanes &= ~lanes_of_row<D>(first);
        visit(first / (D / 4) * (D / 4));
    }
}
__device__ __forceinline__ bool finite(const f32x4 &x) { return cf::finite((x[0] + x[1]) + (x[2] + x[3])); }

template <int D>
__device__ __forceinline__ void f32_fwd_body(const cf_attn_fwd_params &p, int id)
{
    using S = Shape<D>;
    __shared__ f32x4 qs[S::J * 64];
    __shared__ __attribute__((aligned(16))) float parts[NW * S::PART];
    __shared__ float m_s[NW][RB], l_s[NW][RB];
    const int lane = threadIdx.x & 63, wave = wave_id(), quarter = lane >> 4, col = lane & 15;
    const int G = p.n_q_heads / p.n_kv_heads, kh = id % p.n_kv_heads, h = kh * G + id / p.n_kv_heads % G;
    TileLocation loc;
    if (!locate_tile(p.cu_seqlens_q, p.cu_seqlens_k, p.n_segments, p.n_tokens, RB, id / p.n_q_heads, loc)) return;
    const int lq = uniform(loc.len), lk = uniform(loc.other_len), off = lk - lq, q0 = uniform(loc.tile_in_seg) * RB;
    const int rows = min(RB, lq - q0), n_kb = (q0 + rows + off + RB - 1) / RB;
    const float *q = (const float *)p.q + (int64_t)loc.begin * p.q_stride_tok + (int64_t)h * p.q_stride_head;
    const float *k = (const float *)p.k + (int64_t)loc.other_begin * p.kv_stride_tok + (int64_t)kh * p.kv_stride_head;
    const float *v = (const float *)p.v + (int64_t)loc.other_begin * p.kv_stride_tok + (int64_t)kh * p.kv_stride_head;
    const float c2 = p.softmax_scale * kLog2e;
    const unsigned kv_row_bytes = (unsigned)p.kv_stride_tok * 4;
    const int amax = q0 + col + off;                 // last visible key of this lane's row

    f32x4 kf[S::J];
    if (wave < n_kb) load_row<D>(k + (int64_t)min(wave * RB + col, lk - 1) * p.kv_stride_tok, quarter, kf);
    stage_rows<D>(q, p.q_stride_tok, q0, lq - 1, qs);
    __syncthreads();

    Acc<D> o;
#pragma unroll
    for (int x = 0; x < D / 16; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    for (int kb = wave; kb < n_kb; kb += NW) {
        f32x4 x[4][S::NC];
        auto load_v = [&] { load_columns<D>(v + (int64_t)(kb * RB) * p.kv_stride_tok, kv_row_bytes, lk - 1 - kb * RB, lane, x); };
        if (D == 64) load_v();
        f32x4 s = row_product<D>(kf, qs, lane);
        if (D != 64) {
            __builtin_amdgcn_sched_barrier(0);       // V takes the registers of K: with both held D = 128 spills
            load_v();
        }
        if (kb + NW < n_kb) load_row<D>(k + (int64_t)min((kb + NW) * RB + col, lk - 1) * p.kv_stride_tok, quarter, kf);
        const int lim = amax - kb * RB - 4 * quarter;    // key 4 * quarter + i of the block is masked iff i > lim
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = i > lim ? -INFINITY : s[i] * c2;
        const float m_new = fmaxf(m, max_over_quarters(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
        const float ref = m_new == -INFINITY ? 0.f : m_new;     // no visible key yet: every exponential is 0
        const float alpha = __builtin_amdgcn_exp2f(m - ref);
        m = m_new;
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = __builtin_amdgcn_exp2f(s[i] - ref);
        l = l * alpha + ((s[0] + s[1]) + (s[2] + s[3]));
#pragma unroll
        for (int x = 0; x < D / 16; ++x) o[x] *= alpha;
        add_column_product<D>(x, s, o);
    }
    l = sum_over_quarters(l);
    if (quarter == 0) {
        m_s[wave][col] = m;
        l_s[wave][col] = l;
    }
    if (wave < n_kb) write_part<D>(o, parts + wave * S::PART, lane);
    __syncthreads();

    // O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w over the wavefronts that had a block
    const int n = min(NW, n_kb), r = threadIdx.x / (D / 4), c = threadIdx.x % (D / 4);
    bool bad = false;
    if (r < rows) {
        float M = m_s[0][r], L = 0.f;
        for (int w = 1; w < n; ++w) M = fmaxf(M, m_s[w][r]);
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < n; ++w) {
            const float g = __builtin_amdgcn_exp2f(m_s[w][r] - M);
            L += g * l_s[w][r];
            a += g * *(const f32x4 *)(parts + w * S::PART + r * S::OS + c * 4);
        }
        a *= 1.f / L;
        bad = !finite(a);
        *(f32x4 *)((float *)p.o + (int64_t)(loc.begin + q0 + r) * p.o_stride_tok + (int64_t)h * p.o_stride_head + c * 4) = a;
        if (c == 0) p.lse[(int64_t)h * p.n_tokens + loc.begin + q0 + r] = M * kLn2 + logf(L);
    }
    for_rows_of<D>(__ballot(bad), [&](int first) {
        const int row = q0 + (wave * 64 + first) / (D / 4);
        const float *qr = q + (int64_t)row * p.q_stride_tok;
        scalar_fwd_row<float, D, 4>(p, SegmentRows{loc.begin, lq, loc.other_begin, lk}, loc.begin + row, h, [&](int x) { return qr[x]; });
    });
}

template <int D>
__global__ __launch_bounds__(NW * 64) void f32_fwd_kernel(cf_attn_fwd_params p) { f32_fwd_body<D>(p, blockIdx.x); }

// Several chunks in one launch; of a chunk's workgroups the first dkv_blocks[c] belong to its key rows and those of the chunks chained behind
// it.
template <typename Params, int MAX>
struct Batch {
    Blocks<MAX> blocks;
    int dkv_blocks[MAX], next[MAX];
    Params p[MAX];
    bool append(const Params &chunk, int64_t dkv, int64_t others, int next_chunk = -1)
    {
        const int i = blocks.n;
        if (!blocks.append(dkv + others)) return false;
        p[i] = chunk;
        dkv_blocks[i] = (int)dkv;
        next[i] = next_chunk;
        return true;
    }
};
using FwdBatch = Batch<cf_attn_fwd_params, CF_FWD_BATCH_MAX>;
using BwdBatch = Batch<BwdArgs, CF_BWD_BATCH_MAX>;
static_assert(sizeof(BwdBatch) <= 4096 && sizeof(FwdBatch) <= 4096, "kernel arguments");
template <int D>
__global__ __launch_bounds__(NW * 64) void f32_fwd_batch_kernel(FwdBatch q)
{
    int id = blockIdx.x;
    const int c = q.blocks.chunk_of(id);
    f32_fwd_body<D>(q.p[c], id);
}

// exp(s scale - lse).  The scores keep their natural units, in which LSE is exact, and the rounding of the product with log2e
// is put back (e^x = 2^hi (1 + lo ln2)): with both folded into one fma the errors of dQ and dK were a tenth larger than the
// scalar kernels'.
__device__ __forceinline__ float probability(float s, float scale, float lse)
{
    const float x = __builtin_fmaf(s, scale, -lse), hi = x * kLog2e, e = __builtin_amdgcn_exp2f(hi);
    return __builtin_fmaf(e, __builtin_fmaf(x, kLog2e, -hi) * kLn2, e);
}

// dQ of 16 query rows of one head.
template <int D>
__device__ __forceinline__ void f32_dq_body(const BwdArgs &b, int id, char *smem)
{
    using S = Shape<D>;
    const BwdArgs::Fwd &p = b.f;
    f32x4 *qs = (f32x4 *)smem, *dos = (f32x4 *)(smem + S::OPERAND);
    float *del_s = (float *)(smem + 2 * S::OPERAND);
    float *parts = (float *)(smem + S::OPERANDS);    // of each wavefront: its block's keys, in the end its result
    const int lane = threadIdx.x & 63, wave = wave_id(), quarter = lane >> 4, col = lane & 15;
    const int G = p.n_q_heads / p.n_kv_heads, kh = id % p.n_kv_heads, h = kh * G + id / p.n_kv_heads % G;
    TileLocation loc;
    if (!locate_tile(p.cu_seqlens_q, p.cu_seqlens_k, p.n_segments, p.n_tokens, RB, id / p.n_q_heads, loc)) return;
    const int lq = uniform(loc.len), lk = uniform(loc.other_len), off = lk - lq, q0 = uniform(loc.tile_in_seg) * RB;
    const int rows = min(RB, lq - q0), n_kb = (q0 + rows + off + RB - 1) / RB;
    const float *k = (const float *)p.k + (int64_t)loc.other_begin * p.kv_stride_tok + (int64_t)kh * p.kv_stride_head;
    const float *v = (const float *)p.v + (int64_t)loc.other_begin * p.kv_stride_tok + (int64_t)kh * p.kv_stride_head;
    const float *d_o = (const float *)b.d_o + (int64_t)loc.begin * b.do_stride_tok + (int64_t)h * b.do_stride_head;
    const float *o = (const float *)p.o + (int64_t)loc.begin * p.o_stride_tok + (int64_t)h * p.o_stride_head;
    stage_rows<D>((const float *)p.q + (int64_t)loc.begin * p.q_stride_tok + (int64_t)h * p.q_stride_head, p.q_stride_tok, q0, lq - 1, qs);
    stage_rows<D>(d_o, b.do_stride_tok, q0, lq - 1, dos);
    static_assert(NW == RB, "a wavefront forms one row's delta");
    {
        const int r = wave, row = min(q0 + r, lq - 1), c = lane;
        float s = 0.f;
        if (c < D / 4) {
            const f32x4 x = *(const f32x4 *)(d_o + (int64_t)row * b.do_stride_tok + c * 4), y = *(const f32x4 *)(o + (int64_t)row * p.o_stride_tok + c * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_fmaf(x[e], y[e], s);
        }
        for (int x = 32; x > 0; x >>= 1) s += __shfl_xor(s, x);
        if (c == 0) del_s[r] = s;
    }
    const float lse = p.lse[(int64_t)h * p.n_tokens + loc.begin + min(q0 + col, lq - 1)];
    const int amax = q0 + col + off;
    __syncthreads();
    // Rows that see at most 64 keys (large P, large |O|: the rounding of O would be the largest error of dQ) take delta =
    // sum_j P_j dP_j instead.  All rows of the unit then, whose key blocks are one each of the first four wavefronts.
    if (q0 + off + RB <= kExactDeltaKeys) {
        __shared__ float sums[kExactDeltaKeys / RB][RB];
        float sum = 0.f;
        if (wave < n_kb) {
            const int row = min(wave * RB + col, lk - 1);
            f32x4 f[S::J];
            load_row<D>(k + (int64_t)row * p.kv_stride_tok, quarter, f);
            const f32x4 s = row_product<D>(f, qs, lane);
            load_row<D>(v + (int64_t)row * p.kv_stride_tok, quarter, f);
            const f32x4 dp = row_product<D>(f, dos, lane);
            const int lim = amax - wave * RB - 4 * quarter;
#pragma unroll
            for (int i = 0; i < 4; ++i) sum += i > lim ? 0.f : probability(s[i], p.softmax_scale, lse) * dp[i];
            sum = sum_over_quarters(sum);
            if (quarter == 0) sums[wave][col] = sum;
        }
        __syncthreads();
        if (threadIdx.x < RB) {
            float d = sums[0][threadIdx.x];
            for (int w = 1; w < n_kb; ++w) d += sums[w][threadIdx.x];
            del_s[threadIdx.x] = d;
        }
        __syncthreads();
    }
    const float dlt = del_s[col];

    Acc<D> dq;
#pragma unroll
    for (int x = 0; x < D / 16; ++x) dq[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kb = wave; kb < n_kb; kb += NW) {
        const int row = min(kb * RB + col, lk - 1);
        f32x4 kf[S::J], vf[S::J];
        load_row<D>(k + (int64_t)row * p.kv_stride_tok, quarter, kf);
        load_row<D>(v + (int64_t)row * p.kv_stride_tok, quarter, vf);
        put_rows<D>(kf, parts + wave * S::PART, lane);
        const f32x4 s = row_product<D>(kf, qs, lane);
        f32x4 dp = row_product<D>(vf, dos, lane);
        const int lim = amax - kb * RB - 4 * quarter;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float pv = i > lim ? 0.f : probability(s[i], p.softmax_scale, lse);
            dp[i] = pv * (dp[i] - dlt);
        }
        add_column_product<D>(parts + wave * S::PART, lane, dp, dq);
    }
    lds_turn();
    if (wave < n_kb) write_part<D>(dq, parts + wave * S::PART, lane);
    __syncthreads();
    const int n = min(NW, n_kb), r = threadIdx.x / (D / 4), c = threadIdx.x % (D / 4);
    bool bad = false;
    if (r < rows) {
        const f32x4 a = sum_parts<D>(parts, n, r, c) * p.softmax_scale;
        bad = !finite(a);
        *(f32x4 *)((float *)b.d_q + (int64_t)(loc.begin + q0 + r) * b.dq_stride_tok + (int64_t)h * b.dq_stride_head + c * 4) = a;
    }
    for_rows_of<D>(__ballot(bad), [&](int first) {
        const int row = loc.begin + q0 + (wave * 64 + first) / (D / 4);
        const SegmentRows g{loc.begin, lq, loc.other_begin, lk};
        const float *qr = row_of<float>(p.q, row, p.q_stride_tok, h, p.q_stride_head), *dr = row_of<float>(b.d_o, row, b.do_stride_tok, h, b.do_stride_head);
        scalar_dq_row<float, D, 4>(b, g, row, h, [&](int x) { return qr[x]; }, [&](int x) { return dr[x]; }, scalar_delta<float, D>(b, g, row, h));
    });
}

// dK, dV of 16 key rows of one key/value head: (query head of the group, 16-row query block) pairs dealt over the
// wavefronts.
template <int D, bool CHAINS>
__device__ __forceinline__ void f32_dkv_body(const BwdArgs &b, int id, char *smem, float (*stat)[2 * RB])
{
    using S = Shape<D>;
    // In D = 128's kernel of chains dK/dV fills the 128 registers, and what the compiler keeps of the lane from one use to the next, or over
    // a chain of slices, it makes room for by spilling (26 registers, reloaded in the loop over blocks: 3 packed chunks of 532 tokens, 4 heads,
    // 79 us a step, 71 with none; the 4799 tokens above 791 -> 757).
    constexpr bool ANEW = CHAINS && D == 128;
    const BwdArgs::Fwd &p = b.f;
    f32x4 *ks = (f32x4 *)smem, *vs = (f32x4 *)(smem + S::OPERAND);
    float *parts = (float *)(smem + S::OPERANDS);    // of each wavefront: its block's rows, in the end its results
    const int lane = threadIdx.x & 63, wave = wave_id(), quarter = lane >> 4, col = lane & 15;
    const int G = p.n_q_heads / p.n_kv_heads, kh = id % p.n_kv_heads;
    TileLocation loc;
    if (!locate_tile<ANEW>(p.cu_seqlens_k, p.cu_seqlens_q, p.n_segments, p.n_kv_tokens, RB, id / p.n_kv_heads, loc)) return;
    const int lk = uniform(loc.len), lq = uniform(loc.other_len), off = lk - lq;
    // (tiles are numbered from a segment's end; its FIRST key tiles are seen by the most rows: start with those)
    const int k0 = ((lk + RB - 1) / RB - 1 - uniform(loc.tile_in_seg)) * RB, rows = min(RB, lk - k0);
    const int qb_first = max(0, k0 - off) / RB, n_qb = (lq + RB - 1) / RB - qb_first;
    if (n_qb <= 0) return;
    const int n_items = G * n_qb;
    stage_rows<D, ANEW>((const float *)p.k + (int64_t)loc.begin * p.kv_stride_tok + (int64_t)kh * p.kv_stride_head, p.kv_stride_tok, k0, lk - 1, ks);
    stage_rows<D, ANEW>((const float *)p.v + (int64_t)loc.begin * p.kv_stride_tok + (int64_t)kh * p.kv_stride_head, p.kv_stride_tok, k0, lk - 1, vs);
    float *piece = parts + wave * S::PART, *st = stat[wave];                          // this wavefront's LSE and delta by query row
    __syncthreads();

    Acc<D> dk, dv;
#pragma unroll
    for (int x = 0; x < D / 16; ++x) dk[x] = dv[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int n = wave; n < n_items; n += NW) {
        const int row_lane = ANEW ? lane_again<0>(lane, n) : lane, quarter_ = ANEW ? row_lane >> 4 : quarter, col_ = ANEW ? row_lane & 15 : col;
        const int g = n / n_qb, q0 = (qb_first + n - g * n_qb) * RB, h = kh * G + g;
        const float *q = (const float *)p.q + (int64_t)(loc.other_begin + q0) * p.q_stride_tok + (int64_t)h * p.q_stride_head;
        const float *d_o = (const float *)b.d_o + (int64_t)(loc.other_begin + q0) * b.do_stride_tok + (int64_t)h * b.do_stride_head;
        const int last = lq - 1 - q0, row = min(col_, last);      // relative to the block's first row
        // At D = 64 everything an item reads is requested at once (one latency; short calls are made of those); at
        // D = 128 there are registers for one operand at a time.
        f32x4 a[S::J], qa[S::J];
        load_row<D>(d_o + (int64_t)row * b.do_stride_tok, quarter_, a);
        auto load_q_row = [&] { load_row<D>(q + (int64_t)row * p.q_stride_tok, quarter_, qa); };
        if (D == 64) load_q_row();
        const float *orow = (const float *)p.o + (int64_t)(loc.other_begin + q0 + row) * p.o_stride_tok + (int64_t)h * p.o_stride_head;
        float dlt = 0.f;
#pragma unroll
        for (int j = 0; j < S::J; ++j) {
            const f32x4 y = *(const f32x4 *)(orow + 16 * j + 4 * quarter_);
#pragma unroll
            for (int e = 0; e < 4; ++e) dlt = __builtin_fmaf(a[j][e], y[e], dlt);
        }
        dlt = sum_over_quarters(dlt);
        const float lse = p.lse[(int64_t)h * p.n_tokens + loc.other_begin + q0 + row];
        if (quarter_ == 0) {
            st[col_] = col_ <= last ? lse : kNoRow;
            st[RB + col_] = dlt;
        }
        __builtin_amdgcn_wave_barrier();
        put_rows<D>(a, piece, row_lane);
        f32x4 dp = row_product<D>(a, vs, row_lane);
        if (D != 64) load_q_row();
        f32x4 s = row_product<D>(qa, ks, row_lane);
        const int sum_lane = ANEW ? lane_again<1>(lane, n) : lane, q4 = ANEW ? sum_lane >> 4 : quarter, key = ANEW ? sum_lane & 15 : col;
        const int lim = k0 + key - off - q0 - 4 * q4;                // query 4 * q4 + i of the block is masked iff i < lim
        const f32x4 l4 = *(const f32x4 *)(st + 4 * q4);
        f32x4 d4 = *(const f32x4 *)(st + RB + 4 * q4);
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = lim > i ? 0.f : probability(s[i], p.softmax_scale, l4[i]);
        if (q0 + off == 0) {
            // rows that see this key block and no other: delta = sum_j P_j dP_j (as dQ has it for more rows)
#pragma unroll
            for (int i = 0; i < 4; ++i) d4[i] = sum_over_16_lanes(lim > i ? 0.f : s[i] * dp[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) dp[i] = s[i] * (dp[i] - d4[i]);
        __builtin_amdgcn_wave_barrier();                             // st is rewritten by the next item
        add_column_product<D>(piece, sum_lane, s, dv);
        put_rows<D>(qa, piece, sum_lane);
        add_column_product<D>(piece, sum_lane, dp, dk);
    }
    // At D = 64 both results meet in LDS together, at D = 128 there is room for one after the other.
    const int n = min(NW, n_items), end_lane = D == 128 ? fresh_lane() : lane;
    constexpr int TOGETHER = S::BOTH_MEET ? 2 : 1;
    static_assert(TOGETHER * RB * (D / 4) <= NW * 64, "one step");
    const int t = threadIdx.x, r = t / (D / 4) % rows, c = t % (D / 4);
    unsigned long long left_out[2 / TOGETHER];       // lanes whose row is not finite
    for (int first = 0; first < 2; first += TOGETHER) {
        // (what the gradients hold already is fetched while the partial results meet: fetched behind that, steps of 13 small calls, 1 head and 4
        // heads, D = 64, took 45.1 and 46.1 us instead of 44.1 and 44.8, of 3 packed chunks of 600 tokens, 4 heads, D = 128, 88.6 instead of 87.7)
        const int which = TOGETHER == 1 ? first : t / (rows * (D / 4));
        const bool mine = t < TOGETHER * rows * (D / 4);
        f32x4 *to = (f32x4 *)((which ? b.d_k : b.d_v) + (int64_t)(loc.begin + k0 + r) * b.dkv_stride_tok + (int64_t)kh * b.dkv_stride_head + c * 4);
        f32x4 held = {0.f, 0.f, 0.f, 0.f}, a = held;
        if (mine) held = *to;
        if (first == 0) lds_turn();
        else __syncthreads();
        if (wave < n_items) {
            if (first == 0) write_part<D>(dv, parts + wave * S::PART, end_lane);
            if (first + TOGETHER == 2) write_part<D>(dk, parts + ((TOGETHER - 1) * NW + wave) * S::PART, end_lane);
        }
        __syncthreads();
        if (mine) a = sum_parts<D>(parts + (which - first) * NW * S::PART, n, r, c) * (which ? p.softmax_scale : 1.f);
        const unsigned long long bad = __ballot(!finite(a));
        left_out[first / TOGETHER] = bad;
        if (mine && (bad & lanes_of_row<D>(end_lane)) == 0) *to = held + a;
    }
    for (int pass = 0; pass < 2 / TOGETHER; ++pass)
        for_rows_of<D>(left_out[pass], [&](int at) {
            const int first = wave * 64 + at, krow = loc.begin + k0 + first / (D / 4) % rows;
            const bool is_k = (TOGETHER == 1 ? pass : first / (rows * (D / 4))) != 0;
            const SegmentRows g{loc.other_begin, lq, loc.begin, lk};
            const float *kr = row_of<float>(p.k, krow, p.kv_stride_tok, kh, p.kv_stride_head), *vr = row_of<float>(p.v, krow, p.kv_stride_tok, kh, p.kv_stride_head);
            float gk[D / 64], gv[D / 64];
            scalar_dkv_row<float, D, 4>(b, g, krow, kh, [&](int x) { return kr[x]; }, [&](int x) { return vr[x]; },
                                        [&](int row, int h) { return scalar_delta<float, D>(b, g, row, h); }, gk, gv);
            float *dst = (is_k ? b.d_k : b.d_v) + (int64_t)krow * b.dkv_stride_tok + (int64_t)kh * b.dkv_stride_head;
#pragma unroll
            for (int x = 0; x < D / 64; ++x) dst[end_lane + 64 * x] += is_k ? gk[x] * p.softmax_scale : gv[x];
        });
}

template <int D>
struct BwdLds {
    using S = Shape<D>;
    static constexpr int bytes = S::OPERANDS + (S::BOTH_MEET ? 2 : 1) * NW * S::PART * 4;
};
template <int D>
__global__ __launch_bounds__(NW * 64) void f32_bwd_kernel(BwdArgs b, int dkv_blocks)
{
    __shared__ __attribute__((aligned(16))) char smem[BwdLds<D>::bytes];
    __shared__ __attribute__((aligned(16))) float stat[NW][2 * RB];
    const int id = blockIdx.x;
    if (id < dkv_blocks) f32_dkv_body<D, false>(b, id, smem, stat);
    else f32_dq_body<D>(b, id - dkv_blocks, smem);
}
// Slices of one sequence add to the same dK/dV rows.  One workgroup adds to 16 of them for all slices of the launch, slice by
// slice as the calls would, so that a split sequence does not take a launch per slice, each ending with one
// workgroup's chain on a nearly empty chip (the two steps above, a sequence in 3 slices each: 56.0 -> 51.4 us, 928 -> 889).
template <int D>
__global__ __launch_bounds__(NW * 64) void f32_bwd_batch_kernel(BwdBatch q)
{
    __shared__ __attribute__((aligned(16))) char smem[BwdLds<D>::bytes];
    __shared__ __attribute__((aligned(16))) float stat[NW][2 * RB];
    int id = blockIdx.x, c = q.blocks.chunk_of(id);
    if (id >= q.dkv_blocks[c]) {
        f32_dq_body<D>(q.p[c], id - q.dkv_blocks[c], smem);
        return;
    }
    for (;;) {
        f32_dkv_body<D, true>(q.p[c], id, smem, stat);
        c = q.next[c];
        if (c < 0) return;
        __syncthreads();                             // the rows that other wavefronts have written, and LDS
    }
}

// Upper bounds on block counts: sum_g ceil(L_g / 16) <= total / 16 + n_segments.
int64_t row_blocks(int64_t total, int n_segments) { return total / RB + n_segments; }
int64_t query_blocks(const cf_attn_fwd_params &p) { return row_blocks(p.n_tokens, p.n_segments) * p.n_q_heads; }
int64_t key_blocks(const cf_attn_fwd_params &p) { return row_blocks(p.n_kv_tokens, p.n_segments) * p.n_kv_heads; }

int64_t launch_blocks(const cf_attn_fwd_params &p, bool backward) { return query_blocks(p) + (backward ? key_blocks(p) : 0); }

template <int D>
hipError_t run_fwd(const cf_attn_fwd_params &p, hipStream_t s)
{
    const int64_t blocks = launch_blocks(p, false);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const ProfileHook hook = take_profile_hook();
    if (hook.start) (void)hipEventRecord(hook.start, s);
    f32_fwd_kernel<D><<<dim3((unsigned)blocks), NW * 64, 0, s>>>(p);
    const hipError_t e = hipGetLastError();
    if (hook.stop) (void)hipEventRecord(hook.stop, s);
    return e;
}

template <int D>
hipError_t run_bwd(const cf_attn_bwd_params &b, hipStream_t s)
{
    const int64_t dkv = key_blocks(b.f), dq = query_blocks(b.f);
    if (launch_blocks(b.f, true) > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const ProfileHook hook = take_profile_hook();
    if (hook.start) (void)hipEventRecord(hook.start, s);
    f32_bwd_kernel<D><<<dim3((unsigned)(dkv + dq)), NW * 64, 0, s>>>(b, (int)dkv);
    const hipError_t e = hipGetLastError();
    if (hook.stop) (void)hipEventRecord(hook.stop, s);
    return e;
}

}  // namespace

int64_t f32_launch_size(const cf_attn_fwd_params &p, bool backward) { return launch_blocks(p, backward) * NW * 64; }

hipError_t launch_f32_fwd(const cf_attn_fwd_params &p, hipStream_t s) { return p.head_dim == 64 ? run_fwd<64>(p, s) : run_fwd<128>(p, s); }
hipError_t launch_f32_bwd(const cf_attn_bwd_params &b, hipStream_t s) { return b.f.head_dim == 64 ? run_bwd<64>(b, s) : run_bwd<128>(b, s); }

hipError_t launch_f32_fwd_batch(const cf_attn_fwd_params *const *chunks, int n, hipStream_t s)
{
    if (n < 1 || n > CF_FWD_BATCH_MAX) return hipErrorInvalidValue;
    FwdBatch q;
    q.blocks.clear();
    for (int c = 0; c < n; ++c)
        if (!q.append(*chunks[c], 0, query_blocks(*chunks[c]))) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)q.blocks.end);
    if (chunks[0]->head_dim == 64) f32_fwd_batch_kernel<64><<<grid, NW * 64, 0, s>>>(q);
    else f32_fwd_batch_kernel<128><<<grid, NW * 64, 0, s>>>(q);
    return hipGetLastError();
}

hipError_t launch_f32_bwd_batch(const cf_attn_bwd_params *const *chunks, int n, hipStream_t s)
{
    if (n < 1 || n > CF_BWD_BATCH_MAX) return hipErrorInvalidValue;
    const CallChains<CF_BWD_BATCH_MAX> chain(n, [&](int c) -> const cf_attn_bwd_params & { return *chunks[c]; });
    int place[CF_BWD_BATCH_MAX];
    for (int i = 0; i < n; ++i) place[chain.order[i]] = i;
    BwdBatch q;
    q.blocks.clear();
    for (int i = 0; i < n; ++i) {
        const int c = chain.order[i];
        int64_t dkv = 0;                             // a chain's key rows go with its first call: as many as its longest one has
        for (int a = c; chain.head[c] == c && a >= 0; a = chain.next[a]) dkv = std::max(dkv, key_blocks(chunks[a]->f));
        if (!q.append(*chunks[c], dkv, query_blocks(chunks[c]->f), chain.next[c] < 0 ? -1 : place[chain.next[c]])) return hipErrorInvalidConfiguration;
    }
    const dim3 grid((unsigned)q.blocks.end);
    if (chunks[0]->f.head_dim == 64) f32_bwd_batch_kernel<64><<<grid, NW * 64, 0, s>>>(q);
    else f32_bwd_batch_kernel<128><<<grid, NW * 64, 0, s>>>(q);
    return hipGetLastError();
}

}  // namespace cf
