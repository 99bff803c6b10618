// Internal launch interface between the C ABI (api.hip) and the kernel files.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "chunkflow.h"

namespace cf {

// Backward scratch inside the caller's workspace:
//   delta     [Hq][T] fp32: rowsum(dO * O) between the scalar kernels, MINUS that between the bf16 matrix kernels (whose dK/dV
//             kernel starts an accumulator with it)
//   worklist  bf16 MFMA path only: the dK/dV kernel's work items, written by the first workgroups of the dQ launch
//             (layout in attn_mfma_bwd.hip); worklist_items = capacity of its item array
struct BwdWorkspace {
    float *delta;
    int *worklist;
    int64_t worklist_items;
};
// Upper bound on the dK/dV work items of one key/value head (one item = a key tile and some of its (query head, query tile)
// pairs), and the room that the list needs at least (it is cut less finely then).
int64_t dkv_worklist_capacity(const cf_attn_fwd_params &p);
int64_t dkv_worklist_least(const cf_attn_fwd_params &p);

// One-shot event pair recorded around the main kernel of the next launch on this thread (see
// cf_profile_next_call); both NULL when unset.
struct ProfileHook {
    hipEvent_t start = nullptr, stop = nullptr;
};
ProfileHook take_profile_hook();

// Work-items of the largest launch that a call makes on these kernels; one launch holds fewer than 2^32 (a HIP limit).
int64_t f32_launch_size(const cf_attn_fwd_params &p, bool backward);
int64_t mfma_launch_size(const cf_attn_fwd_params &p, bool backward);
int64_t mfma_bwd_blocks(const cf_attn_fwd_params &p);
constexpr int64_t kMostWorkItems = 0xffffffffLL;
// On the scalar kernels, the last resort, where the runtime refuses a call of more: the work-items of the longest row of workgroups, a
// wavefront to a row of Q or of K, to each of the first 64 rows of a segment (delta of the rows with few keys) or to four deltas.
constexpr int kScalarWaves = 4;      // wavefronts per workgroup
inline int64_t simple_launch_size(const cf_attn_fwd_params &p, bool backward)
{
    auto of = [](int64_t wavefronts) { return (wavefronts + kScalarWaves - 1) / kScalarWaves * (kScalarWaves * 64); };
    if (!backward) return of(p.n_tokens);
    return std::max({of(p.n_kv_tokens), of((int64_t)p.n_segments * 64), of(((int64_t)p.n_tokens * p.n_q_heads + 3) / 4)});
}

// fp32 matrix kernels, head_dim 64 and 128; the backward is one launch and needs no scratch.
hipError_t launch_f32_fwd(const cf_attn_fwd_params &p, hipStream_t s);
hipError_t launch_f32_bwd(const cf_attn_bwd_params &p, hipStream_t s);
// Several chunks of one head_dim as one launch (limits as for the bf16 kernels below).  Backward: in the order of the calls, those
// that add to the same rows of d_k / d_v same_key_rows().
hipError_t launch_f32_fwd_batch(const cf_attn_fwd_params *const *chunks, int n, hipStream_t s);
hipError_t launch_f32_bwd_batch(const cf_attn_bwd_params *const *chunks, int n, hipStream_t s);

// What the matrix kernels of the backward read of a call, and what a launch of several calls needs for each of them: 16 of these are a
// kernel's arguments (4096 bytes; of the calls' own structs 14 would fit).  Names as in cf_attn_bwd_params.  A step of 16 packed chunks of
// 512 tokens, 28 / 4 heads, in two backward launches per kernel (8 calls each): 269 us, in one: 234; chunks of 8192: no change.
struct BwdArgs {
    struct Fwd {
        float softmax_scale;
        uint16_t n_q_heads, n_kv_heads;
        int32_t n_tokens, n_kv_tokens, n_segments, n_q_tiles;
        const int32_t *cu_seqlens_q, *cu_seqlens_k;
        const void *q;
        int64_t q_stride_tok, q_stride_head;
        const void *k, *v;
        int64_t kv_stride_tok, kv_stride_head;
        const void *o;
        int64_t o_stride_tok, o_stride_head;
        const float *lse;
        const cf_q_tile *q_tiles;
    } f;
    const void *d_o;
    int64_t do_stride_tok, do_stride_head;
    void *d_q;
    int64_t dq_stride_tok, dq_stride_head;
    float *d_k, *d_v;
    int64_t dkv_stride_tok, dkv_stride_head;

    BwdArgs() = default;
    BwdArgs(const cf_attn_bwd_params &b)
        : f{b.f.softmax_scale, (uint16_t)b.f.n_q_heads, (uint16_t)b.f.n_kv_heads, b.f.n_tokens, b.f.n_kv_tokens, b.f.n_segments, b.f.n_q_tiles,
            b.f.cu_seqlens_q, b.f.cu_seqlens_k, b.f.q, b.f.q_stride_tok, b.f.q_stride_head, b.f.k, b.f.v, b.f.kv_stride_tok,
            b.f.kv_stride_head, b.f.o, b.f.o_stride_tok, b.f.o_stride_head, b.f.lse, b.f.q_tiles},
          d_o(b.d_o), do_stride_tok(b.do_stride_tok), do_stride_head(b.do_stride_head), d_q(b.d_q), dq_stride_tok(b.dq_stride_tok),
          dq_stride_head(b.dq_stride_head), d_k(b.d_k), d_v(b.d_v), dkv_stride_tok(b.dkv_stride_tok), dkv_stride_head(b.dkv_stride_head)
    {
    }
};

// The workgroups of a launch of up to MAX chunks: those of one chunk follow those of the one before it.
template <int MAX>
struct Blocks {
    int n, end;          // chunks, workgroups
    int first[MAX];      // workgroup of each chunk; behind the last one a number that no workgroup has

    void clear()
    {
        n = end = 0;
        std::fill(first, first + MAX, 0x7fffffff);
    }
    bool append(int64_t blocks)
    {
        if (n == MAX || end + blocks > 0x7fffffffLL - MAX) return false;
        first[n++] = end;
        end += (int)blocks;
        return true;
    }
    // The chunk of workgroup id; id becomes its number among the chunk's.  All bounds are read at once: read one by one until the right one
    // was found, they were up to 15 scalar loads in a row at the start of every workgroup (steps of 16 packed chunks of 512 tokens, 28 / 4
    // heads: 217 -> 213 us; of 13 small fp32 calls 45.2 -> 44.6).
    __device__ __forceinline__ int chunk_of(int &id) const
    {
        int c = 0, at = 0;
#pragma unroll
        for (int i = 1; i < MAX; ++i) {
            c = id >= first[i] ? i : c;
            at = id >= first[i] ? first[i] : at;
        }
        id -= at;
        return c;
    }
};

// Order of the calls of a list in a launch that they share, whose workgroups start in that order, for kernels whose workgroups run over
// the keys of some query rows: does a's longest chain of key tiles come before c's (then by queries x keys)?  A launch ends with its
// longest chain, so the chunk that has it goes first, however little work it is.  Of a chunk of several sequences only the mean length is
// known here; the longest is taken for four times that (ten lengths of a lognormal distribution, sigma 0.9), and a prefix is one
// sequence's.  Against the order by queries x keys, us a step: 16 / 4 heads, D = 64, five chunks of 4096 tokens, one of them 904 rows behind
// 4096 keys: 935 -> 758 (compute units idle half of forward and dQ before); 28 / 4 heads, four packed chunks of 2048: 409 -> 384; eight chunks
// of 8192: no change.  Other spreads, 28 / 4 heads, chunks of 2048: all sequences of 500 or all of 100 242.0 and 275.5 either way; one of 1500
// and ten of 50 in every chunk 399.2 and 399.9; D = 64, a sequence of 5000 in slices and thirty of 400 762 -> 573; where the estimate errs, two
// chunks of one of 1800 and six of 40 beside two of four of 500, 369 -> 383.
inline int64_t longest_chain(const cf_attn_fwd_params &p)
{
    const int64_t own = p.n_segments == 1 ? p.n_tokens : std::min<int64_t>(p.n_tokens, 4 * (int64_t)p.n_tokens / p.n_segments);
    return p.n_kv_tokens - p.n_tokens + own;
}
inline int64_t work_of(const cf_attn_fwd_params &p) { return (int64_t)p.n_tokens * p.n_kv_tokens; }
inline bool starts_before(const cf_attn_fwd_params &a, const cf_attn_fwd_params &c)
{
    const int64_t la = longest_chain(a), lc = longest_chain(c);
    return la != lc ? la > lc : work_of(a) > work_of(c);
}

// Single slices whose key row r adds to the same rows of d_k and d_v for every r: key tile t of the one is key tile t of the other.
inline bool same_key_rows(const cf_attn_bwd_params &a, const cf_attn_bwd_params &b)
{
    return a.f.n_segments == 1 && b.f.n_segments == 1 && a.d_k == b.d_k && a.d_v == b.d_v && a.dkv_stride_tok == b.dkv_stride_tok &&
           a.dkv_stride_head == b.dkv_stride_head;
}
// Chains of such calls, each in the order of the calls: where one writer per row adds for all slices of a sequence, these share a
// launch and every workgroup of the chain's first call goes through the chain (which gives the bits of separate launches).
//   head[c]  first call of c's chain        next[c]  the call behind c in it, -1: none
//   order    the calls by the query rows that the first keys of their chain see (of a chunk of several sequences: longest_chain), in steps of
//            512, then by its work (queries x keys), a chain's calls next to each other.  A launch ends with the workgroup of the most rows:
//            16 / 4 heads, D = 64, five chunks of 4096, a sequence in two slices among them: by work alone 748 us a step, so 724; four
//            packed chunks of 4096: 593, 567; where all rows are short, in steps of 1 instead of 512, 1-2 % slower
template <int MAX>
struct CallChains {
    int head[MAX], next[MAX], order[MAX];
    template <typename CallAt>
    CallChains(int n, CallAt call)
    {
        int64_t work[MAX], longest[MAX];
        for (int c = 0; c < n; ++c) {
            head[c] = order[c] = c;
            next[c] = -1;
            work[c] = work_of(call(c).f);
            longest[c] = call(c).f.n_segments == 1 ? call(c).f.n_tokens : longest_chain(call(c).f);
            for (int a = c - 1; a >= 0 && head[c] == c; --a)
                if (same_key_rows(call(a), call(c))) {
                    head[c] = head[a];
                    next[a] = c;
                    work[head[c]] += work[c], longest[head[c]] += longest[c];
                }
        }
        std::stable_sort(order, order + n, [&](int x, int y) {
            const int64_t lx = longest[head[x]] / 512, ly = longest[head[y]] / 512;      // (of the whole chain: its slices may be shorter than a step)
            if (lx != ly) return lx > ly;
            return work[head[x]] != work[head[y]] ? work[head[x]] > work[head[y]] : head[x] < head[y];
        });
    }
};

// Plain scalar kernels: any supported head_dim, fp32 or bf16 storage, fp32 arithmetic.
hipError_t launch_simple_fwd(const cf_attn_fwd_params &p, hipStream_t s);
hipError_t launch_simple_bwd(const cf_attn_bwd_params &p, const BwdWorkspace &ws, hipStream_t s);

// delta[h][t] = sum_d dO[t][h][d] * O[t][h][d].
hipError_t launch_delta(const cf_attn_bwd_params &p, const BwdWorkspace &ws, hipStream_t s);

// head_dim 128, forward and dQ: 32x32x16 MFMAs instead of 16x16x32 (mfma_common.h)?  A launch that fills the chip is limited by power and
// gains 2-7 % from the smaller ones.  On a chip that is mostly empty a wavefront is alone on its SIMD, and the time to issue twice as many
// is added to its chain: forwards of up to 1000 rows behind 3000-50000 keys 3.2-3.7 % slower, backwards 1 %.  What shares a call's launch
// may not decide, since its bits depend on the choice; so the line lies where 16 calls, the most of a launch, have no more workgroups (of 128
// rows and a head) than the chip holds, 512.  8000 tokens of 8 / 2 heads in slices of 512, all forwards in a launch: 228 us with
// 16x16x32, 219 with 32x32x16; in slices of 1000: 160 and 162.
inline bool wide_mfma(const cf_attn_fwd_params &p) { return p.head_dim == 64 || (int64_t)p.n_tokens * p.n_q_heads <= 32 * 128; }

// bf16 MFMA kernels, head_dim 64 and 128 (one head_dim per batch).
hipError_t launch_mfma_fwd(const cf_attn_fwd_params &p, hipStream_t s);
// Forward of 1..CF_FWD_BATCH_MAX chunks as one launch, workgroups dealt in the order of `chunks`.
constexpr int CF_FWD_BATCH_MAX = 16;
hipError_t launch_mfma_fwd_batch(const cf_attn_fwd_params *const *chunks, int n, hipStream_t s);
hipError_t launch_mfma_bwd(const cf_attn_bwd_params &p, const BwdWorkspace &ws, hipStream_t s);
// Backward of 1..CF_BWD_BATCH_MAX (as many as kernel arguments hold) chunks: one dQ launch, then the dK/dV kernels, one launch per
// run of chunks that can share it (run_bwd_batch).
constexpr int CF_BWD_BATCH_MAX = 16;
struct BwdBatchChunk {
    const cf_attn_bwd_params *b;
    BwdWorkspace ws;
    unsigned meets;              // bit a: its d_k / d_v rows may be rows of chunk a before it
};
hipError_t launch_mfma_bwd_batch(const BwdBatchChunk *chunks, int n, hipStream_t s);

}  // namespace cf
