// bf16 MFMA forward kernel for one chunk, head_dim 64 and 128 (paper sections 2.1, 2.2, 4.2: causal mask per
// packed sequence; a dependent chunk's queries also read the retained key/value prefix).
//
// One workgroup = 4 wavefronts; each wavefront owns a unit = 32 consecutive query rows of one query head.  A tile
// of 128 rows and the G query heads of a key/value head make 4 G units, dealt four at a time (block-major) to G
// workgroups: the units of a workgroup share the key/value head and (almost) the key range.  Key/value tiles
// of 64 rows are copied straight from global memory into LDS (buffer loads with an LDS destination, double
// buffered, XOR-swizzled rows) and shared by the four wavefronts.
// Everything is computed TRANSPOSED so that a lane owns one query:
//     S^T = K Q^T   (A = K tile rows from LDS, B = Q^T kept in registers for the whole kernel)
//     O^T += V^T P^T (A = V^T through transposing LDS reads, B = P^T straight from the S^T registers)
// With the query on the lane axis the row maximum and row sum are in-lane reductions plus an exchange between the
// lanes of a query (made only where one of them finds a new maximum), the running rescale is a lane scalar, and P never
// leaves registers.
// Only tiles that intersect the causal diagonal apply a mask; tiles above it are never visited.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "mfma_common.h"
#include "scalar_rows.h"

namespace cf {
namespace {

constexpr int BM = 128;        // query rows per workgroup
constexpr int BN = 64;         // key rows per tile
// Log2 units a row maximum may exceed the running reference before O is rescaled.  D = 64: none, so that no exponent that
// counts is far from zero, where its rounding would be the largest error of the row sum.
template <int D>
constexpr float kLazy = D == 64 ? 0.f : 8.f;

template <int D>
struct Stage {
    static constexpr int tile_bytes = BN * 2 * D;    // one swizzled K or V tile (see mfma_common.h)
    static constexpr int bytes = 2 * tile_bytes;     // K then V
};

// id: index of the workgroup among those of this chunk; SHARED: of several chunks in a launch
// D = 64 keeps what the scalar kernels keep in fp32: the second product takes P with all its 24 bits, as three bf16 operands
// (three MFMAs), exponentials and row sums are formed so that the errors of O and LSE against fp64 are no larger than theirs.
template <int D, int M, bool SHARED>
__device__ __forceinline__ void fwd_body(const cf_attn_fwd_params &p, int id, char *stage_a, char *stage_b)
{
    using F = Mfma<M>;
    constexpr int KS = D / F::K, DB = D / F::M, KB = BN / F::M, QB = F::N32, TILE_BYTES = Stage<D>::tile_bytes;
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int group = F::group(), col = F::column();
    // (Not at D = 128 for a call alone or where M = 32: the main loop then begins 8 or 16 bytes elsewhere in its cache line, which costs
    // long calls more than their start gains, also with the very same registers in the loop.  Calls alone, us, together and now: 28 / 4
    // heads, 250 rows behind 100000 keys 1700 and 1684; 4 / 4, one sequence of 10006 179.1 and 177.3; 14 / 2, 7749 207.7 and 206.9; short
    // calls 0.1 us the other way, 32 / 32, 182 rows 7.6 and 7.7.  M = 32: 8 / 2 heads, 250 rows behind 100000 keys 1642 and 1596.  D = 64,
    // alone: 16 / 4 heads, 4096 packed around 300 19.5 together, 19.9 not; 6 / 2, 500 rows behind 9000 keys 172.7 and 174.0.)
    const RowArgs a(p, D == 64 || (SHARED && M == 16));

    // Block id -> (tile rank, head).  The key/value head varies fastest so that the workgroups an XCD
    // receives (ids are dealt round-robin over the 8 XCDs) keep re-reading the same K/V head in its L2.
    const int G = a.n_q_heads / a.n_kv_heads;
    const int kh = id % a.n_kv_heads;
    id /= a.n_kv_heads;
    const int j = id % G;                            // which of the G workgroups of this (tile, key/value head)
    const int rank = id / G;
    // The tile's 4 G units (32-row block, query head of the group) are dealt out four at a time, block-major:
    // the wavefronts of a workgroup then share at most two neighbouring blocks, so that they need (almost) the
    // same key tiles and a ragged last tile costs workgroups in proportion to its rows.
    const int unit = 4 * j + wave;
    const int blk = unit / G;
    const int h = kh * G + (unit - blk * G);

    int tile_in_seg, q_seg0, lq, k_seg0, lk;
    if (a.tiles != nullptr) {
        if (rank >= a.n_tiles) return;
        const QTile t = read_q_tile(a.tiles, rank);
        tile_in_seg = t.tile_in_seg, q_seg0 = t.q_begin, lq = t.q_len, k_seg0 = t.k_begin, lk = t.k_len;
    } else {
        TileLocation loc;
        if (!locate_tile(p.cu_seqlens_q, p.cu_seqlens_k, p.n_segments, p.n_tokens, BM, rank, loc)) return;
        // (the same in every lane, but values that leave the search loop do not look that way to the compiler)
        tile_in_seg = uniform(loc.tile_in_seg);
        q_seg0 = uniform(loc.begin), lq = uniform(loc.len), k_seg0 = uniform(loc.other_begin), lk = uniform(loc.other_len);
    }
    const int off = lk - lq;                         // prefix keys every row of the segment sees
    const int q_tile0 = tile_in_seg * BM;
    const int rows_valid = min(BM, lq - q_tile0);
    if (q_tile0 + (4 * j) / G * 32 >= lq) return;    // all four units lie beyond the last row
    const int kmax = q_tile0 + min(rows_valid, ((4 * j + 3) / G + 1) * 32) + off;   // keys [0, kmax) are visible to some row of the workgroup
    const int n_tiles = (kmax + BN - 1) / BN;

    const int wq0 = q_tile0 + blk * 32;              // first row of this wavefront (segment-local)
    const int wave_kmax = min(kmax, wq0 + 32 + off); // keys this wavefront needs (<= 0 rows valid: nothing)
    const bool wave_active = wq0 < lq;
    const int amax = wq0 + col + off;                // last visible key of this lane's row (block qb: M qb further)

    const int64_t kv_row_bytes = a.kv_tok * 2;
    const char *kbase = uniform(a.k + ((int64_t)k_seg0 * a.kv_tok + (int64_t)kh * a.kv_head) * 2);
    const char *vbase = uniform(a.v + ((int64_t)k_seg0 * a.kv_tok + (int64_t)kh * a.kv_head) * 2);
    TileDma<BN, D> dma;
    dma.init(kv_row_bytes);

    // Q^T fragments: lane (col, group) holds row wq0 + M*qb + col, d = K*ks + 8*group + 0..7.
    bf16x8 qf[QB][KS];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int row = q_seg0 + min(wq0 + F::M * qb + col, lq - 1);
        const char *qrow = a.q + ((int64_t)row * a.q_tok + (int64_t)h * a.q_head) * 2;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[qb][ks] = *(const bf16x8 *)(qrow + ks * 2 * F::K + group * 16);
    }
    const LaneOffsets<D, M> lo = lane_offsets<D, M>();

    RowBlock<D, M> o_acc;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) o_acc[db][qb] = F::zero();
    // Exponentials: D = 128 in log2 units, the scale folded into them (exp2(s c2 - m), m in those units); D = 64 in the natural
    // units of the scores, exp2((s c2 - m) log2e), where the rounding of log2e only acts on the distance to the maximum.
    constexpr float kLog2e = 1.44269504088896340736f, kUnit = D == 64 ? kLog2e : 1.f;
    const float c2 = p.softmax_scale * (D == 64 ? 1.f : kLog2e);
    float m_run[QB], l_run[QB];                      // running max (those units) and this lane's partial row sum
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) m_run[qb] = -INFINITY, l_run[qb] = 0.f;

    auto issue_tile = [&](int tile_start, char *stage) {
        dma.issue(kbase + (int64_t)tile_start * kv_row_bytes, lk - 1 - tile_start, stage);
        dma.issue(vbase + (int64_t)tile_start * kv_row_bytes, lk - 1 - tile_start, stage + TILE_BYTES);
    };
    issue_tile(0, stage_a);
    wait_lds_dma();
    __syncthreads();

    auto do_tile = [&](int t, const char *stage, char *next_stage) {
        const int tile_start = t * BN;
        if (t + 1 < n_tiles) issue_tile(tile_start + BN, next_stage);

        if (wave_active && tile_start < wave_kmax) {
            // ---- S^T = K Q^T : KB key blocks by QB query blocks
            // All 16 K fragments (D = 128) are requested before the first MFMA: the LDS latency is paid once per tile,
            // not once per MFMA (the matrix unit then consumes them in arrival order).
            typename F::Acc s[KB][QB];
            bf16x8 ka[KB][KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) ka[kb][ks] = lds_read_b128(stage + kb * (TILE_BYTES / KB) + lo.row_unit[ks]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) s[kb][qb] = F::zero();
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int x = 0; x < QB; ++x) {
                        const int qb = kb & 1 ? QB - 1 - x : x;      // (neighbours share an operand)
                        s[kb][qb] = F::mul(ka[kb][ks], qf[qb][ks], s[kb][qb]);
                    }
            // Element i of a query's scores: register i % R of block i / R, key tile_start + place(i) + 4*group.
            constexpr int NS = KB * F::R;
            // ---- causal mask, only on tiles that cross this wavefront's diagonal
            if (tile_start + BN - 1 > wq0 + off) {
                // masked iff the compile-time part of the key exceeds lim (one compare with a constant + one select per element)
                const int lim = amax - tile_start - group * 4;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int i = 0; i < NS; ++i)
                        if (F::place(i) - F::M * qb > lim) s[i / F::R][qb][i % F::R] = -INFINITY;
            }
            // ---- online softmax (log2 domain)
            // Lazy rescale: the running reference m_run only moves when a row's new maximum exceeds it by more than
            // 2^kLazy; until then P = exp2(s - m_run) <= 2^kLazy, exact enough in the fp32 sums and in bf16 alike,
            // and O needs no rescale.  The final division by l_tot and the LSE absorb whatever reference was used.
            // The lanes of a query look at their own keys and meet only where one of them has a new maximum.
            float mx2[QB];
            bool grow = false;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float mx = s[0][qb][0];
#pragma unroll
                for (int i = 1; i < NS; ++i) mx = fmaxf(mx, s[i / F::R][qb][i % F::R]);
                mx2[qb] = mx * c2;
                grow = grow || mx2[qb] > m_run[qb] + kLazy<D>;       // first tile: m_run = -inf
            }
            if (__builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    const float mx = max_over_groups<M>(mx2[qb]), m_new = mx > m_run[qb] + kLazy<D> ? mx : m_run[qb];
                    const float alpha = __builtin_amdgcn_exp2f((m_run[qb] - m_new) * kUnit);   // first tile: exp2(-inf) = 0
                    m_run[qb] = m_new;
                    l_run[qb] *= alpha;
#pragma unroll
                    for (int db = 0; db < DB; ++db) o_acc[db][qb] *= alpha;
                }
            }
            // (the row sum in short chains at D = 64: rounding grows with a chain's length)
            constexpr int CHAINS = D == 64 ? 8 : 1;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float rs[CHAINS] = {};
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i / F::R][qb][i % F::R], c2, -m_run[qb]) * kUnit);
                    s[i / F::R][qb][i % F::R] = pv;
                    rs[i % CHAINS] += pv;
                }
#pragma unroll
                for (int n = CHAINS / 2; n > 0; n /= 2)
#pragma unroll
                    for (int i = 0; i < n; ++i) rs[i] += rs[i + n];
                l_run[qb] += rs[0];
            }
            // ---- O^T += V^T P^T : contraction over the 64 keys in groups of K
            const char *vst = stage + TILE_BYTES;
#pragma unroll
            for (int t = 0; t < BN / F::K; ++t) {
                bf16x8 pb[QB][3];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    float f[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[e] = s[(8 * t + e) / F::R][qb][(8 * t + e) % F::R];
                    if (D == 64) split_exact(f, pb[qb]);
                    else pb[qb][0] = pack8(f);
                }
                const char *va = vst + t * (TILE_BYTES / (BN / F::K));
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const bf16x8 a = lds_read_tr_pair(va + lo.tr_lo[db], va + lo.tr_hi(db));
#pragma unroll
                    for (int x = 0; x < QB; ++x) {
                        const int qb = db & 1 ? QB - 1 - x : x;
#pragma unroll
                        for (int w = 0; w < (D == 64 ? 3 : 1); ++w) o_acc[db][qb] = F::mul(a, pb[qb][w], o_acc[db][qb]);
                    }
                }
            }
        }
        wait_lds_dma();
        __syncthreads();
    };
    for (int t = 0; t < n_tiles; t += 2) {
        do_tile(t, stage_a, stage_b);
        if (t + 1 < n_tiles) do_tile(t + 1, stage_b, stage_a);
    }

    if (!wave_active) return;
    float l_tot[QB], scale[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        l_tot[qb] = sum_over_groups<M>(l_run[qb]);
        scale[qb] = 1.f / l_tot[qb];
    }
    // O rows leave through this wavefront's part of the (now idle) stage buffers, whole rows per store instruction.
    // The scale of a padding row (l_tot = 0 cannot happen: every real row sees its own key) is never stored.
    char *scratch = (wave < 2 ? stage_a : stage_b) + (wave & 1) * RowScratch<D>::bytes;
    store_rows_bf16<D, M>(o_acc, scale, scratch, lq - wq0, [&](int r) {
        return (char *)p.o + ((int64_t)(q_seg0 + wq0 + r) * p.o_stride_tok + (int64_t)h * p.o_stride_head) * 2;
    });
    const int iq = wq0 + (lane & 31);                // lane l < 32 holds the sums of row l, in block l / M
    if (iq < lq && lane < 32) {
        const int qb = QB - 1;
        const float m = lane < F::M ? m_run[0] : m_run[qb], l = lane < F::M ? l_tot[0] : l_tot[qb];
        // One rounding in every kernel: where a product and a sum end up in different blocks, the compiler rounds both.
        p.lse[(int64_t)h * p.n_tokens + q_seg0 + iq] = __builtin_fmaf(m, D == 64 ? 1.f : 0.69314718055994530942f, __logf(l));
    }
    if constexpr (D == 64) {
        for_rows_not_finite<D>(o_acc, scale[0], lq - wq0, [&](int r) {
            const int row = q_seg0 + wq0 + r;
            const unsigned short *qr = row_of<unsigned short>(p.q, row, p.q_stride_tok, h, p.q_stride_head);
            scalar_fwd_row<unsigned short, 64, 4>(p, SegmentRows{q_seg0, lq, k_seg0, lk}, row, h, [&](int x) { return ld(qr + x); });
        });
    }
}

template <int D, int M>
__global__ __launch_bounds__(256, 2) void mfma_fwd_kernel(cf_attn_fwd_params p)
{
    // Two separate arrays (not one array with two halves): the compiler must see that the direct-to-LDS
    // loads of the next tile cannot alias the reads of the current one, or it waits for them too early.
    __shared__ __attribute__((aligned(16))) char stage_a[Stage<D>::bytes];
    __shared__ __attribute__((aligned(16))) char stage_b[Stage<D>::bytes];
    fwd_body<D, M, false>(p, blockIdx.x, stage_a, stage_b);
}

// Several chunks in one launch.  The host
// puts the heaviest chunk first, so the last, partly filled wave of workgroups of a big chunk is filled by
// the next chunk's workgroups instead of leaving compute units idle.
struct FwdBatch {
    unsigned wide;                // bit c: chunk c multiplies with M = 32
    Blocks<CF_FWD_BATCH_MAX> blocks;
    cf_attn_fwd_params p[CF_FWD_BATCH_MAX];
};
// M = 0: chunks with either M.
template <int D, int M>
__global__ __launch_bounds__(256, 2) void mfma_fwd_batch_kernel(FwdBatch b)
{
    __shared__ __attribute__((aligned(16))) char stage_a[Stage<D>::bytes];
    __shared__ __attribute__((aligned(16))) char stage_b[Stage<D>::bytes];
    int id = blockIdx.x;
    const int c = b.blocks.chunk_of(id);
    if (M == 32 || (M == 0 && (b.wide >> c & 1))) fwd_body<D, 32, true>(b.p[c], id, stage_a, stage_b);
    else if constexpr (M != 32) fwd_body<D, 16, true>(b.p[c], id, stage_a, stage_b);
}

// Upper bound on the number of 128-row tiles: sum_g ceil(Lq_g / BM) <= T / BM + n_segments.
int64_t fwd_blocks(const cf_attn_fwd_params &p)
{
    return (p.q_tiles ? (int64_t)p.n_q_tiles : (int64_t)p.n_tokens / BM + p.n_segments) * p.n_q_heads;
}

}  // namespace

int64_t mfma_launch_size(const cf_attn_fwd_params &p, bool backward) { return (backward ? mfma_bwd_blocks(p) : fwd_blocks(p)) * 256; }

hipError_t launch_mfma_fwd_batch(const cf_attn_fwd_params *const *chunks, int n, hipStream_t s)
{
    if (n < 1 || n > CF_FWD_BATCH_MAX) return hipErrorInvalidValue;
    FwdBatch b;
    b.wide = 0;
    b.blocks.clear();
    for (int c = 0; c < n; ++c) {
        b.p[c] = *chunks[c];
        b.wide |= (unsigned)wide_mfma(*chunks[c]) << c;
        if (!b.blocks.append(fwd_blocks(*chunks[c]))) return hipErrorInvalidConfiguration;
    }
    const dim3 grid((unsigned)b.blocks.end);
    if (chunks[0]->head_dim == 64) mfma_fwd_batch_kernel<64, 32><<<grid, 256, 0, s>>>(b);
    else if (b.wide == 0) mfma_fwd_batch_kernel<128, 16><<<grid, 256, 0, s>>>(b);
    else if (b.wide == (1u << n) - 1) mfma_fwd_batch_kernel<128, 32><<<grid, 256, 0, s>>>(b);
    else mfma_fwd_batch_kernel<128, 0><<<grid, 256, 0, s>>>(b);
    return hipGetLastError();
}

hipError_t launch_mfma_fwd(const cf_attn_fwd_params &p, hipStream_t s)
{
    const int64_t blocks = fwd_blocks(p);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const ProfileHook hook = take_profile_hook();
    if (hook.start) (void)hipEventRecord(hook.start, s);
    const dim3 grid((unsigned)blocks);
    if (p.head_dim == 64) mfma_fwd_kernel<64, 32><<<grid, 256, 0, s>>>(p);
    else if (wide_mfma(p)) mfma_fwd_kernel<128, 32><<<grid, 256, 0, s>>>(p);
    else mfma_fwd_kernel<128, 16><<<grid, 256, 0, s>>>(p);
    const hipError_t e = hipGetLastError();
    if (hook.stop) (void)hipEventRecord(hook.stop, s);
    return e;
}

}  // namespace cf
