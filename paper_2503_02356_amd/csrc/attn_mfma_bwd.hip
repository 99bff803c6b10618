// bf16 MFMA backward kernels for one chunk, head_dim 64 and 128 (paper section 4.2: key/value gradients of the
// retained prefix rows are accumulated by the later chunks' backward passes; section 2.2: per-sequence
// causal mask inside a packed chunk).
//
// Two kernels, no dQ atomics:
//
//  dkv kernel  A workgroup (4 wavefronts) owns 128 (D = 64: 32) consecutive key rows of one segment, a wavefront 32 of them:
//              their dV^T and dK^T (fp32) and K, V operands stay in its registers for the whole kernel.  It loops over
//              the 64-row (D = 64: 128-row) query tiles that can see its keys, for one or several query heads of its
//              key/value head; Q and dO tiles go straight from global memory into two XOR-swizzled LDS stages (row
//              reads and transposing reads are both free of bank conflicts).
//              FUSED_HEADS = true : one workgroup per key tile and key/value head loops over ALL query heads
//                  of the group and is the only writer of its dK/dV rows (plain read-modify-write, bitwise
//                  reproducible).  Used when the launch has enough key tiles to fill the GPU, and always at D = 64.
//              FUSED_HEADS = false: a work list built on the device cuts the (key tile, query heads) work into
//                  items of similar length, longest first; the items of one key/value head meet in dK/dV
//                  through fp32 atomic adds (once per workgroup, at the end).
//
//  dq kernel   Same shape as the forward kernel: a workgroup owns four units of 32 query rows and a head, key/value
//              tiles of 64 rows go through LDS, everything transposed so that a lane owns one query:
//                  S^T = K Q^T   dP^T = V dO^T   dS^T = P^T (dP^T - delta)   dQ^T += K^T dS^T
//              LSE and delta are one scalar per lane; dS^T feeds the last product straight from registers.
//              It also computes delta = <dO, O> (which the dK/dV kernel, launched after it, reads).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "mfma_common.h"
#include "scalar_rows.h"

namespace cf {
namespace {

constexpr float kLog2e = 1.44269504088896340736f;

// =====================================================================================================
// dK / dV
// =====================================================================================================
// How the four wavefronts of a workgroup divide its work: KW groups of 32 keys, QW wavefronts each.
// D = 128: 128 keys per workgroup, whose wavefronts read the same query tiles; query heads are split over work items where that fills
// the chip, through atomic adds.
// D = 64: every dK/dV row has one writer, so no workgroup may share its keys with another: few keys shorten the chain that one workgroup
// is.  The four wavefronts take the 32-row blocks of all the group's heads in turn, one each, and add up in LDS at the end, in a fixed
// order.  No two of them read the same rows, so that each copies its own into its own part of LDS (OWN) and waits for nobody until
// the end.  Steps, us, against tiles of 128 rows of a head that the four copied together, with a barrier for each (wavefronts without rows
// at a head's end waited there): 16 / 4 heads, five chunks of 4096 686 -> 675; 8 / 2 heads, 4500 tokens in slices of 2048 and 3 packed
// chunks 405 -> 394; 6 / 2 heads, 2700 in slices of 1000 and 3 packed chunks 225 -> 218; one head, 700 in slices of 256 60.2 -> 58.8.
// (Eight wavefronts to 32 keys, one workgroup a compute unit, halve the chain: calls of one slice take 4-25 % less, packed chunks 2-10 %
// more, since short sequences leave half of them idle.  By a rule on the call, as the bits have to follow from it alone, a step's slices and
// packed chunks need a launch each, and that costs more than it gives: 705 -> 743, 401 -> 403, 219 -> 219, 58.6 -> 66.0.
// 64 or 128 keys took 4-30 % longer than 32, split heads with atomic adds 4 % less.)
template <int D>
struct DkvShape {
    static constexpr int KW = D == 64 ? 1 : 4, QW = 4 / KW;
    static constexpr int BKV = 32 * KW;               // key rows per workgroup
    static constexpr bool OWN = QW > 1;               // every wavefront has tiles of its own
    static constexpr int BQ = OWN ? 32 : 64;          // query rows per tile
    static constexpr int BLOCKS = BQ / 32;
};
constexpr int BQ = DkvShape<128>::BQ, BKV = DkvShape<128>::BKV;

// ---- work list of the dK/dV kernel (not used in the fused mode) -------------------------------------------
// One item = (segment, key tile, range of its (head of the group, query tile) pairs, head by head): the workgroups of one
// key/value head.  A key tile seen by few query tiles keeps all its pairs in ONE item (one prologue, one epilogue, one set of
// atomic updates); one with more is cut into equal items.  Where the cuts lie:
//   A launch ends with its longest item.  A workgroup that has a compute unit to itself takes 2.2 us per pair, one of two 3.6,
//   so an item of 1.6 times what a workgroup slot gets on average (512 slots, `slots` of them when several chunks share a
//   launch) still ends with the rest, and every item more costs a prologue and an epilogue (some 14 us of its slot).
//   - 1.6 averages <= kFineMost pairs (few rounds of items): items of that many pairs.
//   - Beyond (long sequences, whose items end evenly anyway, and whose extra atomic updates cost more than they balance):
//     whole heads, items of half the average but at most kSplitTarget pairs, except where a head has more than 1.6 averages.
//   - A lone call with an average of at most kSmallMost pairs: 2.2 averages, so that its items are about one for each of
//     the 256 compute units.
//   - Where single heads of key tiles are about one for each compute unit (over 128, up to 256 in such a call), or one to
//     one and a half rounds of all slots, they are the items, as long as they are not much longer than that: their different
//     lengths fill the launch better than equal ones.  Heads of up to three query tiles are never cut.
// dK/dV of one call, us, against items of half the average of whole heads: 28 / 4 heads, 8192 tokens packed around 600: 145
// (196; 1.0 / 2.0 averages: 177 / 147); 4 / 4 heads, 4000 tokens in one sequence: 70 (147); 32 / 8 heads, 2048 tokens packed
// around 200: 43 (71; 1.6 averages: 51); 64 / 8 heads, 500 tokens in one sequence: 37 (37; 1.6 / 2.2 averages: 50 / 41).
// The list is ordered by DESCENDING duration (pairs; a counting sort): workgroups start in list order, and starting the
// longest first is what keeps the last compute units from running one long item alone.
// Workspace layout (ints): [0] = number of items, [64 ...] = the items; an item is int4 {segment, kt0, first pair, pairs}.
constexpr int kSlots = 512, kSplitTarget = 48, kFineMost = 64, kSmallMost = 8;
constexpr int kDurationBuckets = 256;

// sum over segments of ceil(Lk / 128) <= n_kv_tokens / 128 + n_segments
__host__ __device__ inline int64_t key_tiles_most(const cf_attn_fwd_params &p) { return (int64_t)p.n_kv_tokens / BKV + p.n_segments; }
// Items cut inside heads: one per key tile and, beyond that, as many as one key/value head's pairs hold 1.6 / kSlots of all pairs
// (2.2: fewer).  Whole heads: G per key tile.
__host__ __device__ inline int64_t dkv_items_most(const cf_attn_fwd_params &p)
{
    const int64_t tiles = key_tiles_most(p), G = p.n_q_heads / p.n_kv_heads, cuts = kSlots * 10 / 16 / p.n_kv_heads + 1;
    return tiles * G > tiles + cuts ? tiles * G : tiles + cuts;
}

// The rule above, for a call of `total` (key tile, query tile) pairs of a query head in n_tiles key tiles.
struct ListCuts {
    float average;                                   // pairs per slot
    int fair, target;
    bool large, small, even_heads;
    __host__ __device__ ListCuts(int total, int n_tiles, int n_q_heads, int slots)
    {
        const int64_t all_pairs = (int64_t)total * n_q_heads;
        // (in floating point: a rounding moves a cut, and no more; 64-bit divisions would take longer than the rest of the list)
        average = (float)all_pairs / (float)slots;
        const int fine = share(average, 1.6f);
        large = fine > kFineMost, small = slots == kSlots && average <= kSmallMost;
        fair = small ? max(3, share(average, 2.2f)) : fine;
        const int64_t head_items = (int64_t)n_tiles * n_q_heads;
        even_heads = small ? head_items > kSlots / 4 && head_items <= kSlots / 2
                           : !large && head_items > kSlots && head_items <= kSlots * 3 / 2;
        target = max(2, large || even_heads ? (int)fminf(kSplitTarget, average / 2) : fine);
    }
    __host__ __device__ static int share(float average, float averages) { return (int)fminf(ceilf(average * averages), 1e9f); }
    // Items of a key tile that n_qt query tiles see.  heads: of whole query heads (of G).  cut_heads: items may end inside one.
    __host__ __device__ int items(int n_qt, int G, bool cut_heads, bool &heads) const
    {
        const int pairs = G * n_qt, by_heads = min(G, (pairs + target - 1) / target), fairly = (pairs + fair - 1) / fair;
        heads = !cut_heads || (large ? fairly <= by_heads : n_qt <= 3 || (even_heads && n_qt <= (small ? fair * 8 / 5 : fair)));
        return heads ? by_heads : fairly;
    }
};

// Runs in ONE workgroup of 256 threads: among the first of the dQ launch, which the dK/dV kernel follows anyway (no launch
// of its own).
// Segment bounds pass through LDS 256 at a time (one coalesced load instead of a chain of dependent ones); a wavefront
// takes every fourth segment, its lanes the key tiles.
__device__ __forceinline__ void build_dkv_worklist(const BwdArgs::Fwd &p, int *wl, int capacity, int slots)
{
    __shared__ int bucket[kDurationBuckets];        // items per duration, then the next free slot of each duration
    __shared__ int seg_lq[256], seg_lk[256];
    __shared__ int n_items, total, n_tiles;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    bucket[tid] = 0;
    if (tid == 0) total = n_tiles = 0;
    const int G = p.n_q_heads / p.n_kv_heads;
    auto for_each_tile = [&](auto &&visit) {
        for (int base = 0; base < p.n_segments; base += 256) {
            const int n = min(256, p.n_segments - base);
            __syncthreads();
            if (tid < n) {
                seg_lq[tid] = p.cu_seqlens_q[base + tid + 1] - p.cu_seqlens_q[base + tid];
                seg_lk[tid] = p.cu_seqlens_k[base + tid + 1] - p.cu_seqlens_k[base + tid];
            }
            __syncthreads();
            for (int s = wave; s < n; s += 4) {
                const int lq = seg_lq[s], lk = seg_lk[s], off = lk - lq;
                for (int kt0 = lane * BKV; kt0 < lk; kt0 += 64 * BKV) {
                    const int n_qt = (lq + BQ - 1) / BQ - max(0, kt0 - off) / BQ;
                    if (n_qt > 0) visit(base + s, kt0, n_qt);
                }
            }
        }
    };
    int mine = 0, my_tiles = 0;
    for_each_tile([&](int, int, int n_qt) { mine += n_qt, ++my_tiles; });
    atomicAdd(&total, mine);
    atomicAdd(&n_tiles, my_tiles);
    __syncthreads();
    const ListCuts cuts(total, n_tiles, p.n_q_heads, slots);
    bool cut_heads = true;
    auto for_each_item = [&](auto &&visit) {
        for_each_tile([&](int seg, int kt0, int n_qt) {
            bool heads;
            const int sp = cuts.items(n_qt, G, cut_heads, heads);
            // equal shares of the heads or of the pairs, the first few with one more
            const int whole = heads ? G : G * n_qt, unit = heads ? n_qt : 1;
            const int base = sp == 1 ? whole : whole / sp, longer = whole - base * sp;
            for (int s = 0; s < sp; ++s) {
                const int n = (base + (s < longer)) * unit;
                visit(i32x4{seg, kt0, (s * base + min(s, longer)) * unit, n}, min(n, kDurationBuckets - 1));
            }
        });
    };
    for (;;) {
        for_each_item([&](i32x4, int duration) { atomicAdd(&bucket[duration], 1); });
        __syncthreads();
        if (tid == 0) {                              // longest first: slots are handed out from the top bucket down
            int next = 0;
            for (int d = kDurationBuckets - 1; d >= 0; --d) {
                const int n = bucket[d];
                bucket[d] = next;
                next += n;
            }
            n_items = next;
        }
        __syncthreads();
        if (n_items <= capacity || !cut_heads) break;
        cut_heads = false;                           // (at most G items per key tile: what every scratch has room for)
        __syncthreads();
        bucket[tid] = 0;                             // (for_each_item's first barrier comes before its first visit)
    }
    i32x4 *items = (i32x4 *)(wl + 64);
    for_each_item([&](i32x4 item, int duration) {    // (its first barrier comes after the slots are laid out)
        const int slot = atomicAdd(&bucket[duration], 1);
        if (slot < capacity) items[slot] = item;     // (it always is: a scratch has room for G items per key tile)
    });
    if (tid == 0) wl[0] = min(n_items, capacity);
}

// One stage: Q tile, dO tile, LSE[64] (log2 units), -delta[64] (the dQ kernel stores it negated); OWN: one for each wavefront.  Two stages
// (OWN: a wavefront's part of the first) also hold the end-of-kernel transpose scratch (32 rows of D floats per wavefront).
template <int D>
struct DkvStage {
    static constexpr int BQ = DkvShape<D>::BQ;
    static constexpr bool OWN = DkvShape<D>::OWN;
    static constexpr int tile_bytes = BQ * 2 * D, one = 2 * tile_bytes + 2 * 64 * 4, bytes = DkvShape<D>::QW * one;
    static constexpr int scratch_bytes = 32 * D * 4;
    static_assert(OWN ? one >= scratch_bytes : bytes >= 2 * scratch_bytes, "wavefronts turn their results around in a stage");
};

// As RowArgs (mfma_common.h), for this kernel.
struct KeyArgs {
    const char *k, *v, *q, *d_o;
    const int32_t *cu_q, *cu_k;
    int64_t kv_tok, kv_head, q_tok, q_head, do_tok, do_head;
    int n_q_heads, n_kv_heads;
    const int *wl;
    // together: not in chains, which have no registers to keep them in; there each is loaded where it is used.
    __device__ __forceinline__ KeyArgs(const BwdArgs &b, const int *worklist, bool together)
        : kv_tok(b.f.kv_stride_tok), kv_head(b.f.kv_stride_head), q_tok(b.f.q_stride_tok), q_head(b.f.q_stride_head), do_tok(b.do_stride_tok),
          do_head(b.do_stride_head), n_q_heads(b.f.n_q_heads), n_kv_heads(b.f.n_kv_heads)
    {
        auto k_ = (const CF_GLOBAL char *)b.f.k, v_ = (const CF_GLOBAL char *)b.f.v, q_ = (const CF_GLOBAL char *)b.f.q, do_ = (const CF_GLOBAL char *)b.d_o;
        auto cu_q_ = (const CF_CONSTANT int32_t *)b.f.cu_seqlens_q, cu_k_ = (const CF_CONSTANT int32_t *)b.f.cu_seqlens_k;
        auto wl_ = (const CF_CONSTANT int *)worklist;
        if (together)
            asm("" : "+s"(k_), "+s"(v_), "+s"(q_), "+s"(do_), "+s"(cu_q_), "+s"(cu_k_), "+s"(kv_tok), "+s"(kv_head), "+s"(q_tok), "+s"(q_head),
                     "+s"(do_tok), "+s"(do_head), "+s"(n_q_heads), "+s"(n_kv_heads), "+s"(wl_));
        k = (const char *)k_, v = (const char *)v_, q = (const char *)q_, d_o = (const char *)do_;
        cu_q = (const int32_t *)cu_q_, cu_k = (const int32_t *)cu_k_, wl = (const int *)wl_;
    }
};

// A wavefront owns 32 key rows: K_w, V_w (operands) and dV_w^T, dK_w^T (fp32) stay in its
// registers for the whole kernel, 192 of them at D = 128.  Per 32-row block of queries:
//     S = Q K_w^T    P = exp2(S c - LSE)    dP' = dO V_w^T - delta (the accumulator starts at -delta)    dS = P dP'
//     dV_w^T += dO^T P      dK_w^T += Q^T dS
// (A operands from LDS rows resp. transposing LDS reads; lane = key, so P and dS are B operands where they stand).
// Two workgroups share a compute unit, one wavefront of each on a SIMD, with nothing to wait for in each other: while
// one multiplies the other does its arithmetic.
// RESIDUAL tile pairs (those made of a sequence's first 128 positions: query rows at positions < 128 x key tile 0) feed the
// MFMAs the bf16 values of P and dS AND their bf16 rounding residuals: rows that see few keys have large P and dS, whose
// rounding would be the largest error in dK/dV.  At D = 64 P and dS enter every product with all their 24 bits instead, as
// three bf16 operands.
// RING: operand fragments in flight (below).  wave: of this wavefront.
template <int D, bool FUSED_HEADS, int RING = 4>
__device__ __forceinline__ void dkv_body(const BwdArgs &b, const float *__restrict__ delta, int id,
                                         const int *__restrict__ wl, char *st0, char *st1, int wave = wave_id())
{
    using Stage = DkvStage<D>;
    constexpr int M = D == 64 ? 32 : 16;
    using F = Mfma<M>;
    constexpr int KS = D / F::K, DB = D / 32, N = F::N32, BLOCK = 32 * 2 * D;
    constexpr int QW = DkvShape<D>::QW, BQ = DkvShape<D>::BQ, BKV = DkvShape<D>::BKV;
    constexpr bool OWN = DkvShape<D>::OWN;
    static_assert(FUSED_HEADS || QW == 1, "atomic updates are made by the wavefront that owns the keys");
    const BwdArgs::Fwd &p = b.f;
    const int key_wave = wave / QW, query_wave = wave % QW;

    // Block id -> (item, key/value head); the key/value head varies fastest (XCD L2 locality, see forward).
    //   fused mode : item = key tile rank, all G heads of the group
    //   otherwise  : item = entry of the work list
    const KeyArgs first(b, wl, RING != 3);
    auto args = [&] { return RING == 3 ? KeyArgs(b, wl, false) : first; };
    const int G = args().n_q_heads / args().n_kv_heads;
    const int kh = id % args().n_kv_heads;
    id /= args().n_kv_heads;
    int kt0, first_pair = 0, n_pairs = 0, q_seg0, lq, k_seg0, lk;
    // (all of this is the same in every lane, but values that leave locate_tile's search loop do not look that way to
    // the compiler: say so, or everything derived from them lives in vector registers.)
    if (FUSED_HEADS) {
        TileLocation loc;
        if (!locate_tile<RING == 3>(args().cu_k, args().cu_q, p.n_segments, p.n_kv_tokens, BKV, id, loc)) return;
        q_seg0 = uniform(loc.other_begin), lq = uniform(loc.other_len), k_seg0 = uniform(loc.begin), lk = uniform(loc.len);
        // locate_tile numbers tiles from the end; the FIRST key tiles of a segment are seen by the most rows, so
        // flip the order inside the segment to start the heaviest tiles first.
        kt0 = uniform(((loc.len + BKV - 1) / BKV - 1 - loc.tile_in_seg) * BKV);
    } else {
        // (the item and the count at once: there is room for an item of every workgroup)
        const i32x4 item = ((const i32x4 *)(args().wl + 64))[id];
        int n_items = args().wl[0], seg = item[0];
        kt0 = item[1], first_pair = item[2], n_pairs = item[3];
        asm("" : "+s"(n_items), "+s"(seg), "+s"(kt0), "+s"(first_pair), "+s"(n_pairs));
        if (id >= n_items) return;
        int q_seg1 = args().cu_q[seg + 1], k_seg1 = args().cu_k[seg + 1];
        q_seg0 = args().cu_q[seg], k_seg0 = args().cu_k[seg];
        asm("" : "+s"(q_seg0), "+s"(q_seg1), "+s"(k_seg0), "+s"(k_seg1));        // (at once)
        lq = q_seg1 - q_seg0, lk = k_seg1 - k_seg0;
    }
    const int off = lk - lq;
    const int qt_first = max(0, kt0 - off) / BQ;     // first query tile with a row that sees any key of this tile
    const int qt_end = (lq + BQ - 1) / BQ;
    if (qt_first >= qt_end) return;                  // whole workgroup leaves before any barrier
    if (FUSED_HEADS) n_pairs = G * (qt_end - qt_first);
    // (head, query tile) pairs, head by head; OWN: this wavefront's, every QW-th
    const int n_tiles = OWN ? (n_pairs - query_wave + QW - 1) / QW : n_pairs;
    int head_first = FUSED_HEADS ? 0 : first_pair / (qt_end - qt_first), qt_start = qt_first + first_pair - head_first * (qt_end - qt_first);
    auto go_on = [&](int &qt, int &h, int by) {      // to the pair that is `by` further
        qt += by;
        while (qt >= qt_end) qt -= qt_end - qt_first, ++h;
    };
    if (OWN) {
        go_on(qt_start, head_first, query_wave);
        st0 += query_wave * Stage::one, st1 += query_wave * Stage::one;
    }
    // query tiles below qt_head are RESIDUAL ones for this key tile
    const int qt_head = kt0 == 0 && off < 128 ? (128 - off + BQ - 1) / BQ : 0;

    const int kw0 = kt0 + 32 * key_wave;                 // first key of this wavefront (segment-local)
    const bool wave_active = kw0 < lk;
    const float c2 = scalar(p.softmax_scale * kLog2e);

    // B operands kept for the whole kernel: lane = key row, 8 consecutive d per step.
    bf16x8 kf[N][KS], vf[N][KS];
#pragma unroll
    for (int kb = 0; kb < N; ++kb) {
        const int64_t from = ((k_seg0 + min(kw0 + F::M * kb + F::column(), lk - 1)) * args().kv_tok + (int64_t)kh * args().kv_head) * 2 + F::group() * 16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            kf[kb][ks] = *(const bf16x8 *)(args().k + from + ks * 2 * F::K);
            vf[kb][ks] = *(const bf16x8 *)(args().v + from + ks * 2 * F::K);
        }
    }
    f32x16 dv[DB], dk[DB];                           // 32 x 32 blocks: lane % 32 = key, register group j = d 32 db + 8 j + 4 half + 0..3
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) dv[i][j] = dk[i][j] = 0.f;
    BlockAddress<D, M> at;                              // of the block in use

    // Tile staging: Q and dO rows, LSE and -delta go straight from global memory into an LDS stage; once they have landed,
    // wavefront 0 (OWN: each) turns LSE into log2 units (+inf for rows past the segment, so that P = 0).  What the copies need of the
    // lane is made anew per tile: every register counts (a spilled one would be reloaded behind the copies in flight,
    // and the wait for it would be a wait for them).
    int nx_h = kh * G + head_first, nx_qt = qt_start;            // the tile the next copy fetches (advances by additions only)
    auto issue_tile = [&](char *stage) {
        const int h = nx_h, q0 = nx_qt * BQ, lane_ = fresh_lane();
        const int64_t row0 = q_seg0 + q0;
        TileDma<BQ, D, OWN ? 1 : 4, true> dma;
        dma.init(args().q_tok * 2, OWN ? 0 : wave, lane_);
        dma.issue(uniform(args().q + (row0 * args().q_tok + (int64_t)h * args().q_head) * 2), lq - 1 - q0, stage);
        dma.init(args().do_tok * 2, OWN ? 0 : wave, lane_);
        dma.issue(uniform(args().d_o + (row0 * args().do_tok + (int64_t)h * args().do_head) * 2), lq - 1 - q0,
                  stage + Stage::tile_bytes);
        // LSE and -delta of 64 rows (OWN: the tile's and what lies behind them in the segment)
        auto issue_stats = [&](const float *from, int which) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(TileDma<64, D>::descriptor((const char *)uniform(from + (int64_t)h * p.n_tokens + row0)),
                                                     (CF_LDS void *)(stage + 2 * Stage::tile_bytes + which * 256), 4,
                                                     min(lane_, lq - 1 - q0) * 4, 0, 0, 0);
        };
        if (OWN) {
            issue_stats(p.lse, 0);
            issue_stats(delta, 1);
            go_on(nx_qt, nx_h, QW);
        } else {
            if (wave < 2) issue_stats(wave < 1 ? p.lse : delta, wave);
            if (++nx_qt == qt_end) {
                nx_qt = qt_first;
                ++nx_h;
            }
        }
    };
    auto finish_tile = [&](char *stage, int rows) {  // rows: of the segment, in this tile
        wait_lds_dma();
        if (OWN || wave == 0) {
            const int row = fresh_lane();
            float *l = (float *)(stage + 2 * Stage::tile_bytes) + row;
            *l = row < rows ? *l * kLog2e : INFINITY;
        }
    };
    auto publish_tile = [] {
        if (OWN) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        else __syncthreads();
    };
    if (!OWN || n_tiles > 0) {
        issue_tile(st0);
        finish_tile(st0, lq - qt_start * BQ);
    }
    publish_tile();

    int cur_qt = qt_start;                           // query tile of the stage in use
    auto do_block = [&](int mb, const char *stage, bool residual) {
        const int q0 = cur_qt * BQ + mb * 32;
        if (q0 + 31 + off < kw0 || q0 >= lq) return;     // no row of the block sees a key of this wavefront, or none is a row
        const char *qs = stage, *dos = stage + Stage::tile_bytes;
        const float *stats = (const float *)(stage + 2 * Stage::tile_bytes) + mb * 32 + fresh_lane() / F::M * 4;
        // The A operands of the block's four products pass through a ring of fragments, each requested RING uses
        // before its own: ROWS fragments of Q rows and of dO rows, then the transposed dO and Q operands (contraction over the
        // 32 query rows in 2 groups of 16).
        constexpr int ROWS = N * KS, COLS = 2 * DB;
        bf16x8 ring[RING];
        auto fetch = [&](int n) {
            if (n == ROWS || (n >= 2 * ROWS && n % DB == 0)) at.forget();
            if (n < 2 * ROWS) {
                const int m = n % ROWS;
                ring[n % RING] = lds_read_b128((n < ROWS ? qs : dos) + m % N * (BLOCK / N) + at.row(m / N));
            } else if (n < 2 * ROWS + 2 * COLS) {
                const int m = n - 2 * ROWS, db = m % DB, tq = m % COLS / DB;
                const char *rows = (m / COLS ? qs : dos) + tq * (BLOCK / 2);
                ring[n % RING] = lds_read_tr_pair(rows + at.tr_lo(db), rows + at.tr_hi(db));
            }
        };
#pragma unroll
        for (int n = 0; n < RING; ++n) fetch(n);
        // [query block][key block]; element i of a key block: register i % R of query block i / R, query row q0 + place(i) + 4*group
        typename F::Acc s[N][N], dp[N][N];
        constexpr int NS = N * F::R;
#pragma unroll
        for (int qb = 0; qb < N; ++qb)
#pragma unroll
            for (int kb = 0; kb < N; ++kb) s[qb][kb] = F::zero();
#pragma unroll
        for (int n = 0; n < ROWS; ++n) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < N; ++kb) s[n % N][kb] = F::mul(ring[n % RING], kf[kb][n / N], s[n % N][kb]);
            fetch(n + RING);
        }
#pragma unroll
        for (int i = 0; i < NS; i += 4) {
            const f32x4 d4 = *(const f32x4 *)(stats + 64 + F::place(i));
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int kb = 0; kb < N; ++kb) dp[i / F::R][kb][i % F::R + j] = d4[j];
        }
#pragma unroll
        for (int n = ROWS; n < 2 * ROWS; ++n) {
            __builtin_amdgcn_sched_barrier(0);
            const int m = n - ROWS;
#pragma unroll
            for (int kb = 0; kb < N; ++kb) dp[m % N][kb] = F::mul(ring[n % RING], vf[kb][m / N], dp[m % N][kb]);
            fetch(n + RING);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NS; i += 4) {
            const f32x4 l4 = *(const f32x4 *)(stats + F::place(i));
#pragma unroll
            for (int kb = 0; kb < N; ++kb)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    s[i / F::R][kb][i % F::R + j] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i / F::R][kb][i % F::R + j], c2, -l4[j]));
        }
        // The causal mask: selects only on a block that crosses the diagonal (its last key lies after its first query).
        if (kw0 + 31 - off - q0 > 0) {
            const int lane_ = fresh_lane();
            const int lim = kw0 + lane_ % F::M - off - q0 - lane_ / F::M * 4;     // masked iff lim > the constant part of the row
#pragma unroll
            for (int kb = 0; kb < N; ++kb)
#pragma unroll
                for (int i = 0; i < NS; ++i) s[i / F::R][kb][i % F::R] = lim > F::place(i) - F::M * kb ? 0.f : s[i / F::R][kb][i % F::R];
        }
#pragma unroll
        for (int qb = 0; qb < N; ++qb)
#pragma unroll
            for (int kb = 0; kb < N; ++kb)
#pragma unroll
                for (int i = 0; i < F::R; ++i) dp[qb][kb][i] *= s[qb][kb][i];
        // B operand of dV_w^T += dO^T P (x = 0) resp. dK_w^T += Q^T dS for the contraction over query rows 16 tq + 0..15, lane % 32 =
        // key: the bf16 values, or (rest) their rounding residuals.  D = 64: k-slot 8*half + e is row 16 tq + place(e) + 4*half, where
        // the values stand.  D = 128: a quarter q of the lanes has rows 4 q + 0..3 of both key blocks and keeps those of block
        // q % 2; the other quarter of its half gets the other ones for its own: k-slot 8*half + e is row 16 tq + 8*half + e.
        auto value = [&](int x, int i, int kb) { return (x ? dp : s)[i / F::R][kb][i % F::R]; };
        auto operand = [&](int x, int tq, auto rest) {
            bf16x8 w;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float f = N == 1 ? value(x, 8 * tq + e, 0) : value(x, 4 * tq + e % 4, e / 4);
                if (decltype(rest)::value) {
                    asm volatile("" : "+v"(f));      // (the roundings here are not to be kept for the products below)
                    f -= (float)(__bf16)f;
                }
                w[e] = (__bf16)f;
            }
            if (N == 2) {
                i32x4 u = __builtin_bit_cast(i32x4, w);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const u32x2 r = __builtin_amdgcn_permlane16_swap((unsigned)u[i], (unsigned)u[2 + i], false, false);
                    u[i] = (int)r[0], u[2 + i] = (int)r[1];
                }
                w = __builtin_bit_cast(bf16x8, u);
            }
            return w;
        };
        if (D != 64 && residual) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int tq = 0; tq < 2; ++tq) {
                    __builtin_amdgcn_sched_barrier(0);
                    const bf16x8 w = operand(x, tq, std::true_type());
                    const char *rows = (x ? qs : dos) + tq * (BLOCK / 2);
                    at.forget();
#pragma unroll
                    for (int j = 0; j < DB; ++j)
                        accumulate_in_place<D>(x ? dk[j] : dv[j], lds_read_tr_pair(rows + at.tr_lo(j), rows + at.tr_hi(j)), w);
                }
        }
        // Each operand is made right before its use (all four at once: 4 registers too many); D = 64 splits it in three.
        bf16x8 w, ws[3];
#pragma unroll
        for (int m = 0; m < 2 * COLS; ++m) {
            __builtin_amdgcn_sched_barrier(0);
            const int j = m % DB, g = m / DB, x = g / 2, n = 2 * ROWS + m;
            if (D != 64 && j == 0) w = operand(x, g % 2, std::false_type());
            if (D == 64) {
                if (j == 0) {
                    float f[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[e] = value(x, (8 * (g % 2) + e) % NS, 0);
                    split_exact(f, ws);
                }
#pragma unroll
                for (int t = 0; t < 3; ++t) accumulate_in_place<D>(x ? dk[j] : dv[j], ring[n % RING], ws[t]);
            } else {
                accumulate_in_place<D>(x ? dk[j] : dv[j], ring[n % RING], w);
            }
            fetch(n + RING);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto do_tile = [&](int t, const char *stage, char *next_stage) {
        if (t + 1 < n_tiles) issue_tile(next_stage);
        if (wave_active) {
            const bool residual = cur_qt < qt_head;
#pragma unroll 1
            for (int i = 0; i < DkvShape<D>::BLOCKS; ++i) {
                do_block(i, stage, residual);
                if (DkvShape<D>::BLOCKS == 2) at.flip(BLOCK);
            }
        }
        if (OWN) {
            int h = 0;
            go_on(cur_qt, h, QW);
        } else if (++cur_qt == qt_end) {
            cur_qt = qt_first;
        }
        if (t + 1 < n_tiles) finish_tile(next_stage, lq - cur_qt * BQ);
        publish_tile();
    };
    for (int t = 0; t < n_tiles; t += 2) {
        do_tile(t, st0, st1);
        if (t + 1 < n_tiles) do_tile(t + 1, st1, st0);
    }

    // dK, dV: lane = key row; register group g4 of accumulator j = 4 consecutive d starting at 32*j + 8*g4 + 4*half.
    // Each wavefront turns its 32 x D blocks around in LDS (unit u of row r at u ^ (r & 15)) and then updates whole rows, 64 lanes = 64
    // consecutive floats: a lane-per-row update would touch 64 cache lines per instruction.  The room for it is the wavefront's half of a
    // stage, free after the loop's last barrier; OWN: its own part of the first stage, which no other wavefront touches before meet(), and
    // which it has read for the last time itself.
    //   FUSED_HEADS : this workgroup is the only writer of these rows in this launch: plain load, add, store.
    //   otherwise   : the query heads of a group add into the same rows: fp32 atomic adds.
    // QW > 1: the partial results of a key group's wavefronts are added in their order, each of them writes every QW-th group of 8 rows.
    const int rows_valid = min(32, lk - kw0);        // <= 0: this wavefront has no real keys
    if (QW == 1 && rows_valid <= 0) return;
#pragma unroll
    for (int j = 0; j < DB; ++j) {
        accumulator_done(dv[j]);
        accumulator_done(dk[j]);
    }
    auto scratch_of = [&](int w) {
        return (float *)(OWN ? st0 + (w - query_wave) * Stage::one : (w < 2 ? st0 : st1) + (w & 1) * Stage::scratch_bytes);
    };
    auto meet = [] {
        if (QW == 1) __builtin_amdgcn_wave_barrier();
        else __syncthreads();
    };
    float *tr = scratch_of(wave);
    const int end_lane = fresh_lane(), end_half = end_lane >> 5, end_col = end_lane & 31;
    unsigned not_finite[2] = {0, 0};                 // rows of dV and dK that this wavefront has left out (D = 64; see scalar_rows.h)
    auto add_rows = [&](const f32x16 (&acc)[DB], float scale, float *g, unsigned &left_out) {
        float *const rows = g + ((int64_t)(k_seg0 + kw0) * b.dkv_stride_tok + (int64_t)kh * b.dkv_stride_head);
        // FUSED_HEADS: what 8 rows hold already is fetched together, for the first 8 while the results are turned around.  (Row by row, behind
        // each one's test, it was a latency for each of the 64 rows of dV and dK.  Steps, us: 32 / 32 heads, 4000 tokens in slices of 512 and 2
        // packed chunks 873 -> 774; 8 / 8 heads, 20000 in slices of 1000 4165 -> 3933; 16 / 4 heads, D = 64, five chunks of 4096 731 -> 718.)
        float held[8][D / 64];
        auto fetch_held = [&](int r0) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int c = 0; c < D / 64; ++c) held[e][c] = rows[(int64_t)min(r0 + e, rows_valid - 1) * b.dkv_stride_tok + end_lane + 64 * c];
        };
        if (FUSED_HEADS && rows_valid > 8 * query_wave) fetch_held(8 * query_wave);
#pragma unroll
        for (int j = 0; j < DB; ++j)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                f32x4 a;
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = acc[j][g4 * 4 + e] * scale;
                *(f32x4 *)(tr + end_col * D + (((j * 8 + g4 * 2 + end_half) ^ (end_col & 15)) << 2)) = a;
            }
        meet();
        // 8 rows per step: all LDS reads first, then the global updates (one LDS latency per step)
        for (int r0 = 8 * query_wave; r0 < rows_valid; r0 += 8 * QW) {
            float v[8][D / 64];
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int c = 0; c < D / 64; ++c) {
                    const int at_ = (r0 + e) * D + (((16 * c + (end_lane >> 2)) ^ ((r0 + e) & 15)) << 2) + (end_lane & 3);
                    v[e][c] = scratch_of(key_wave * QW)[at_];
#pragma unroll
                    for (int w = 1; w < QW; ++w) v[e][c] += scratch_of(key_wave * QW + w)[at_];
                }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool leave = D == 64 && __ballot(!finite(v[e][0])) != 0;
                if (leave && r0 + e < rows_valid) left_out |= 1u << (r0 + e);
                if (!leave && r0 + e < rows_valid) {
                    float *row = rows + (int64_t)(r0 + e) * b.dkv_stride_tok + end_lane;
#pragma unroll
                    for (int c = 0; c < D / 64; ++c) {
                        if (FUSED_HEADS) row[64 * c] = held[e][c] + v[e][c];
                        else unsafeAtomicAdd(row + 64 * c, v[e][c]);
                    }
                }
            }
            if (FUSED_HEADS && r0 + 8 * QW < rows_valid) fetch_held(r0 + 8 * QW);
        }
        meet();
    };
    add_rows(dv, 1.f, b.d_v, not_finite[0]);
    add_rows(dk, p.softmax_scale, b.d_k, not_finite[1]);
    if (D == 64) {
        for (unsigned rows = not_finite[0] | not_finite[1]; rows != 0; rows &= rows - 1) {
            const int r = __builtin_ctz(rows), krow = k_seg0 + kw0 + r;
            const unsigned short *kr = row_of<unsigned short>(p.k, krow, p.kv_stride_tok, kh, p.kv_stride_head);
            const unsigned short *vr = row_of<unsigned short>(p.v, krow, p.kv_stride_tok, kh, p.kv_stride_head);
            float gk[1], gv[1];
            scalar_dkv_row<unsigned short, 64, 4>(b, SegmentRows{q_seg0, lq, k_seg0, lk}, krow, kh, [&](int x) { return ld(kr + x); },
                                               [&](int x) { return ld(vr + x); },
                                               [&](int row, int h) { return -delta[(int64_t)h * p.n_tokens + row]; }, gk, gv);
            const int64_t at = (int64_t)krow * b.dkv_stride_tok + (int64_t)kh * b.dkv_stride_head + end_lane;
            if (not_finite[0] >> r & 1) b.d_v[at] += gv[0];
            if (not_finite[1] >> r & 1) b.d_k[at] += gk[0] * p.softmax_scale;
        }
    }
}

template <int D, bool FUSED_HEADS>
__global__ __launch_bounds__(256, 2) void mfma_dkv_kernel(BwdArgs b, const float *__restrict__ delta, const int *__restrict__ wl)
{
    // Separate arrays (not one array with parts): the compiler must see that the direct-to-LDS copy of a coming
    // tile cannot alias the reads of the tile in use, or it waits for the copy too early.
    __shared__ __attribute__((aligned(16))) char st0[DkvStage<D>::bytes];
    __shared__ __attribute__((aligned(16))) char st1[DkvStage<D>::bytes];
    dkv_body<D, FUSED_HEADS>(b, delta, blockIdx.x, wl, st0, st1);
}

// Several chunks' backward in one launch.
struct BwdBatch {
    unsigned wide;                                               // bit c: chunk c's dQ multiplies with M = 32
    Blocks<CF_BWD_BATCH_MAX> blocks;
    int next[CF_BWD_BATCH_MAX];                                  // chunk whose dK/dV rows are done behind this one's, by the same workgroups
    int capacity[CF_BWD_BATCH_MAX], slots[CF_BWD_BATCH_MAX];     // of the work list that is built (see there)
    float *delta[CF_BWD_BATCH_MAX];
    int *wl[CF_BWD_BATCH_MAX];                                   // nullptr: no list (one workgroup per key tile)
    BwdArgs b[CF_BWD_BATCH_MAX];
};
static_assert(sizeof(BwdBatch) <= 4096, "kernel arguments");

// Chunks with work lists: they follow each other, each longest first, and the last workgroups of one chunk run beside the first of
// the next.  CHAINS: chunks of disjoint dK/dV rows and chains of slices that add to the same ones, one workgroup to a row: D = 64, 16 / 4
// heads, 16.7k tokens, a sequence in 2 slices: 1014 -> 979 us a step (a launch per slice before); D = 128: run_bwd_batch.  (D = 128
// has one register less then, and four to a fragment.)
template <int D, bool CHAINS>
__global__ __launch_bounds__(256, 2) void mfma_dkv_batch_kernel(BwdBatch q)
{
    __shared__ __attribute__((aligned(16))) char st0[DkvStage<D>::bytes];
    __shared__ __attribute__((aligned(16))) char st1[DkvStage<D>::bytes];
    const int wave = wave_id();
    int id = blockIdx.x, c = q.blocks.chunk_of(id);
    for (;;) {
        if constexpr (D == 128 && CHAINS) dkv_body<D, true, 3>(q.b[c], q.delta[c], id, nullptr, st0, st1, wave);
        else dkv_body<D, CHAINS>(q.b[c], q.delta[c], id, q.wl[c], st0, st1);
        if (!CHAINS) return;
        c = q.next[c];
        if (c < 0) return;
        __syncthreads();                             // LDS has been read for the last time
    }
}

// =====================================================================================================
// dQ
// =====================================================================================================
constexpr int BM = 128;                      // query rows per workgroup
constexpr int BN = 64;                       // key rows per tile
template <int D>
struct KvStage {
    static constexpr int tile_bytes = BN * 2 * D;    // one swizzled K or V tile
    static constexpr int bytes = 2 * tile_bytes;
};

// A workgroup whose 128-row tile starts a sequence (rows at positions < 128: a "head" tile) feeds the dQ product the
// bf16 rounding residual of dS besides dS, as the dK/dV kernel does for these rows (at D = 64 every workgroup feeds it all
// 24 bits of dS, as three operands).  It also replaces delta of its rows: delta = <dO, O> is computed from the ROUNDED O, and for rows that see few keys
// (large P, large |O|) that rounding would be the largest error of the whole backward pass (it lands in dK
// of the first keys of each sequence).  It first runs over its (at most 4) key tiles once to form delta = sum_j P_j dP_j,
// which needs no O, stores it for the dK/dV kernel, then runs again for dQ.
// (A run-time flag, uniform over the workgroup: one code path keeps one register allocation.)
// Short sequences are made of head tiles and bound by what a workgroup does besides multiplying: they are dealt out like
// the others (one query head per workgroup left the wavefronts without rows idle), the second run takes one or two key tiles from
// LDS, where the first has left them, and no tile's second half is computed where no row sees it.  Steps of 16 packed chunks, 28 / 4
// heads: 512 tokens around 37 each 297 -> 269 us, 8192 around 600 9.31 -> 9.05 ms; 16 / 4 heads, D = 64, 16.7k tokens 979 -> 940 us.
template <int D, int M>
__device__ __forceinline__ void dq_body(const BwdArgs &b, float *__restrict__ delta, int id, char *stage_a, char *stage_b)
{
    using F = Mfma<M>;
    constexpr int KS = D / F::K, DB = D / F::M, N = F::N32, KVTILE_BYTES = KvStage<D>::tile_bytes;
    const BwdArgs::Fwd &p = b.f;
    const int wave = wave_id(), group = F::group(), col = F::column();
    // (calls alone, us, against arguments loaded where they are used: 28 / 4 heads, 512 packed around 37 37.2 -> 36.4; 14 / 2, 1747 around 73
    // 51.6 -> 50.9; 28 / 4, 8192 around 600 227.0 -> 227.5; long ones within 0.3 %)
    const RowArgs a(p);

    const int G = a.n_q_heads / a.n_kv_heads;
    const int kh = id % a.n_kv_heads;
    id /= a.n_kv_heads;
    const int j = id % G;                            // which of the G workgroups of this (tile, key/value head)
    const int rank = id / G;

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
    const int off = lk - lq;
    const int q_tile0 = tile_in_seg * BM;
    const bool head = q_tile0 + off < 128;
    // The tile's 4 G units (32-row block, query head of the group) are dealt out four at a time, block-major (as in the
    // forward kernel).
    const int unit = 4 * j + wave;
    const int blk = unit / G;
    const int h = kh * G + (unit - blk * G);
    const int rows_valid = min(BM, lq - q_tile0);
    if (q_tile0 + (4 * j) / G * 32 >= lq) return;    // all four units lie beyond the last row
    const int kmax = q_tile0 + min(rows_valid, ((4 * j + 3) / G + 1) * 32) + off;   // keys [0, kmax) are visible to some row of the workgroup
    const int n_tiles = (kmax + BN - 1) / BN;
    const int wq0 = q_tile0 + blk * 32;
    const int wave_kmax = min(kmax, wq0 + 32 + off);
    const bool wave_active = wq0 < lq;
    const int amax = wq0 + col + off;                // last visible key of this lane's row (block qb: M qb further)

    const int64_t kv_row_bytes = a.kv_tok * 2;
    const char *kbase = uniform(a.k + ((int64_t)k_seg0 * a.kv_tok + (int64_t)kh * a.kv_head) * 2);
    const char *vbase = uniform(a.v + ((int64_t)k_seg0 * a.kv_tok + (int64_t)kh * a.kv_head) * 2);
    TileDma<BN, D, 4, true> dma;
    dma.init(kv_row_bytes);

    // Q^T and dO^T fragments (B operands): lane holds row wq0 + M*qb + col, d = K*ks + 8*group + 0..7
    bf16x8 qf[N][KS], dof[N][KS];
    float lse2[N], dlt[N];
    auto row_of_block = [&](int qb) { return wq0 + F::M * qb + col; };
    auto stat_at = [&](int qb) { return (int64_t)h * p.n_tokens + q_seg0 + min(row_of_block(qb), lq - 1); };
#pragma unroll
    for (int qb = 0; qb < N; ++qb) {
        const int iq = row_of_block(qb), row = q_seg0 + min(iq, lq - 1);
        const char *qrow = a.q + ((int64_t)row * a.q_tok + (int64_t)h * a.q_head) * 2;
        const char *dorow = (const char *)b.d_o + ((int64_t)row * b.do_stride_tok + (int64_t)h * b.do_stride_head) * 2;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qf[qb][ks] = *(const bf16x8 *)(qrow + ks * 2 * F::K + group * 16);
            dof[qb][ks] = *(const bf16x8 *)(dorow + ks * 2 * F::K + group * 16);
        }
        lse2[qb] = iq < lq ? p.lse[stat_at(qb)] * kLog2e : INFINITY;   // padding rows: P = 0
        // delta = <dO, O> of this lane's row (section 4.2's backward needs it for dS): the lanes of a row sum D * M / 64 d each.
        // Published for the dK/dV kernel; head tiles replace it below.
        dlt[qb] = 0.f;
        if (!head) {
            const char *orow = (const char *)p.o + ((int64_t)row * p.o_stride_tok + (int64_t)h * p.o_stride_head) * 2;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 of = *(const bf16x8 *)(orow + ks * 2 * F::K + group * 16);
#pragma unroll
                for (int e = 0; e < 8; ++e) dlt[qb] = __builtin_fmaf((float)of[e], (float)dof[qb][ks][e], dlt[qb]);
            }
            dlt[qb] = sum_over_groups<M>(dlt[qb]);
            if (iq < lq && group == 0) delta[stat_at(qb)] = -dlt[qb];
        }
    }
    const float c2 = p.softmax_scale * kLog2e;
    const LaneOffsets<D, M> lo = lane_offsets<D, M>();

    RowBlock<D, M> dq;
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int qb = 0; qb < N; ++qb) dq[i][qb] = F::zero();

    auto issue_tile = [&](int tile_start, char *stage) {
        dma.issue(kbase + (int64_t)tile_start * kv_row_bytes, lk - 1 - tile_start, stage);
        dma.issue(vbase + (int64_t)tile_start * kv_row_bytes, lk - 1 - tile_start, stage + KVTILE_BYTES);
    };

    // One sweep over the key tiles.  DELTA_PASS: only accumulate sum_j P_j dP_j (this lane's keys) in dsum.
    // staged: how many tiles stand in the stages already.  (One or two tiles are all still there after a first sweep.)
    float dsum[N] = {};
    auto sweep = [&](auto delta_pass_tag, int staged) {
        constexpr bool DELTA_PASS = decltype(delta_pass_tag)::value;
        if (staged == 0) {
            issue_tile(0, stage_a);
            wait_lds_dma();
            __syncthreads();
        }
        auto do_tile = [&](int t, const char *stage, char *next_stage) {
            const int tile_start = t * BN;
            const char *ks_ = stage;
            const char *vs_ = stage + KVTILE_BYTES;
            if (t + 1 < n_tiles && t + 1 >= staged) issue_tile(tile_start + BN, next_stage);

            if (wave_active && tile_start < wave_kmax) {
                const bool need_mask = tile_start + BN - 1 > wq0 + off;
                // element i of a query (register i % R of key block i / R) is key tile_start + 32*mb + place(i) + 4*group:
                // masked iff the compile-time part of that exceeds lim
                const int lim = amax - tile_start - group * 4;
                constexpr int NS = N * F::R;
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    if (mb == 1 && tile_start + 32 >= wave_kmax) break;      // no row sees the second half
                    // S^T and dP^T for 32 keys.
                    // All 16 fragments are requested before the first MFMA: the LDS latency is paid once per
                    // block, not once per MFMA.
                    typename F::Acc s[N][N], dp[N][N];           // [key block][query block]
                    bf16x8 ka[N][KS], va[N][KS];
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int kb = 0; kb < N; ++kb) {
                            const int at = mb * (KVTILE_BYTES / 2) + kb * (KVTILE_BYTES / 2 / N) + lo.row_unit[ks];
                            ka[kb][ks] = lds_read_b128(ks_ + at);
                            va[kb][ks] = lds_read_b128(vs_ + at);
                        }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int kb = 0; kb < N; ++kb)
#pragma unroll
                        for (int qb = 0; qb < N; ++qb) s[kb][qb] = dp[kb][qb] = F::zero();
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int kb = 0; kb < N; ++kb) {
#pragma unroll
                            for (int qb = 0; qb < N; ++qb) s[kb][qb] = F::mul(ka[kb][ks], qf[qb][ks], s[kb][qb]);
                            // (M = 32: S and dP are one chain each; two MFMAs of a chain in a row would wait.  LDS reads may pass.)
                            if (M == 32) __builtin_amdgcn_sched_barrier(0x180);
#pragma unroll
                            for (int qb = 0; qb < N; ++qb) dp[kb][qb] = F::mul(va[kb][ks], dof[qb][ks], dp[kb][qb]);
                            if (M == 32) __builtin_amdgcn_sched_barrier(0x180);
                        }
                    // K^T fragments of the dQ contraction: requested now, so that they arrive during the arithmetic
                    bf16x8 kt[32 / F::K][DB];
                    if (!DELTA_PASS) {
#pragma unroll
                        for (int tq = 0; tq < 32 / F::K; ++tq)
#pragma unroll
                            for (int j = 0; j < DB; ++j) {
                                const char *ka_ = ks_ + mb * (KVTILE_BYTES / 2) + tq * (F::K * 2 * D);
                                kt[tq][j] = lds_read_tr_pair(ka_ + lo.tr_lo[j], ka_ + lo.tr_hi(j));
                            }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (!need_mask) {
#pragma unroll
                        for (int qb = 0; qb < N; ++qb)
#pragma unroll
                            for (int i = 0; i < NS; ++i) {
                                const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i / F::R][qb][i % F::R], c2, -lse2[qb]));
                                if (DELTA_PASS) dsum[qb] += pv * dp[i / F::R][qb][i % F::R];
                                else dp[i / F::R][qb][i % F::R] = pv * (dp[i / F::R][qb][i % F::R] - dlt[qb]);
                            }
                    } else
#pragma unroll
                    for (int qb = 0; qb < N; ++qb)
#pragma unroll
                        for (int i = 0; i < NS; ++i) {
                            float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i / F::R][qb][i % F::R], c2, -lse2[qb]));
                            const bool hidden = need_mask && mb * 32 + F::place(i) - F::M * qb > lim;
                            if (hidden) pv = 0.f;
                            // (dP of a hidden pair may be anything)
                            if (DELTA_PASS) dsum[qb] += D == 64 && hidden ? 0.f : pv * dp[i / F::R][qb][i % F::R];
                            else dp[i / F::R][qb][i % F::R] = pv * (dp[i / F::R][qb][i % F::R] - dlt[qb]);
                        }
                    if (DELTA_PASS) continue;
                    // dQ^T += K^T dS^T : contraction over these 32 keys in groups of K
#pragma unroll
                    for (int tq = 0; tq < 32 / F::K; ++tq) {
                        bf16x8 dsb[N][3];
                        float f[N][8];
#pragma unroll
                        for (int qb = 0; qb < N; ++qb) {
#pragma unroll
                            for (int e = 0; e < 8; ++e) f[qb][e] = dp[(8 * tq + e) / F::R][qb][(8 * tq + e) % F::R];
                            if (D == 64) split_exact(f[qb], dsb[qb]);
                            else dsb[qb][0] = pack8(f[qb]);
                        }
#pragma unroll
                        for (int x = 0; x < (D == 64 ? 3 : 1); ++x)
#pragma unroll
                            for (int j = 0; j < DB; ++j)
#pragma unroll
                                for (int n = 0; n < N; ++n) {
                                    const int qb = j & 1 ? N - 1 - n : n;    // (neighbours share an operand)
                                    dq[j][qb] = F::mul(kt[tq][j], dsb[qb][x], dq[j][qb]);
                                }
                        if (D != 64 && head) {   // add the bf16 rounding residual of dS
                            bf16x8 dl[N];
#pragma unroll
                            for (int qb = 0; qb < N; ++qb)
#pragma unroll
                                for (int e = 0; e < 8; ++e) dl[qb][e] = (__bf16)(f[qb][e] - (float)dsb[qb][0][e]);
#pragma unroll
                            for (int j = 0; j < DB; ++j)
#pragma unroll
                                for (int qb = 0; qb < N; ++qb) dq[j][qb] = F::mul(kt[tq][j], dl[qb], dq[j][qb]);
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
    };
    if (head) {
        sweep(std::true_type(), 0);
#pragma unroll
        for (int qb = 0; qb < N; ++qb) {
            dlt[qb] = sum_over_groups<M>(dsum[qb]);  // the lanes of a row hold different keys of it
            if (row_of_block(qb) < lq && group == 0) delta[stat_at(qb)] = -dlt[qb];
        }
    }
    sweep(std::false_type(), head && n_tiles <= 2 ? n_tiles : 0);

    if (wave_active) {
        // dQ rows leave through this wavefront's part of the (now idle) stage buffers, whole rows per store instruction
        char *scratch = (wave < 2 ? stage_a : stage_b) + (wave & 1) * RowScratch<D>::bytes;
        float scale[N];
#pragma unroll
        for (int qb = 0; qb < N; ++qb) scale[qb] = p.softmax_scale;
        store_rows_bf16<D, M>(dq, scale, scratch, lq - wq0, [&](int r) {
            return (char *)b.d_q + ((int64_t)(q_seg0 + wq0 + r) * b.dq_stride_tok + (int64_t)h * b.dq_stride_head) * 2;
        });
        if constexpr (D == 64) {
            for_rows_not_finite<D>(dq, p.softmax_scale, lq - wq0, [&](int r) {
                const int row = q_seg0 + wq0 + r;
                const unsigned short *qr = row_of<unsigned short>(p.q, row, p.q_stride_tok, h, p.q_stride_head);
                const unsigned short *dr = row_of<unsigned short>(b.d_o, row, b.do_stride_tok, h, b.do_stride_head);
                scalar_dq_row<unsigned short, 64, 4>(b, SegmentRows{q_seg0, lq, k_seg0, lk}, row, h, [&](int x) { return ld(qr + x); },
                                                  [&](int x) { return ld(dr + x); }, __shfl(dlt[0], r));
            });
        }
    }
}

// wl != nullptr: the launch has one extra workgroup (the first) that builds the dK/dV work list.
template <int D, int M>
__global__ __launch_bounds__(256, 2) void mfma_dq_kernel(BwdArgs b, float *__restrict__ delta, int *wl, int capacity)
{
    // The list builder is workgroup 0: it starts with the first wave of workgroups and is long done when the
    // launch ends (as the last workgroup it would start last and could be what the launch ends with).
    if (D == 128 && wl != nullptr && blockIdx.x == 0) {
        build_dkv_worklist(b.f, wl, capacity, kSlots);
        return;
    }
    // Two separate arrays (not one array with two halves): the compiler must see that the direct-to-LDS
    // loads of the next tile cannot alias the reads of the current one, or it waits for them too early.
    __shared__ __attribute__((aligned(16))) char stage_a[KvStage<D>::bytes];
    __shared__ __attribute__((aligned(16))) char stage_b[KvStage<D>::bytes];
    dq_body<D, M>(b, delta, (int)blockIdx.x - (wl != nullptr ? 1 : 0), stage_a, stage_b);
}

// Several chunks, heaviest first: dQ and delta of a chunk depend on nothing another chunk's backward writes, so the last,
// partly filled wave of workgroups of a big chunk can be filled by the next chunk's.  The first q.n workgroups build the
// chunks' dK/dV work lists.
// M = 0: chunks with either M.
template <int D, int M>
__global__ __launch_bounds__(256, 2) void mfma_dq_batch_kernel(BwdBatch q)
{
    int id = (int)blockIdx.x - q.blocks.n;
    if (id < 0) {
        const int c = blockIdx.x;
        if (D == 128 && q.wl[c] != nullptr) build_dkv_worklist(q.b[c].f, q.wl[c], q.capacity[c], q.slots[c]);
        return;
    }
    __shared__ __attribute__((aligned(16))) char stage_a[KvStage<D>::bytes];
    __shared__ __attribute__((aligned(16))) char stage_b[KvStage<D>::bytes];
    const int c = q.blocks.chunk_of(id);
    if (M == 32 || (M == 0 && (q.wide >> c & 1))) dq_body<D, 32>(q.b[c], q.delta[c], id, stage_a, stage_b);
    else if constexpr (M != 32) dq_body<D, 16>(q.b[c], q.delta[c], id, stage_a, stage_b);
}

// Launch geometry of one chunk's backward.
struct BwdShape {
    bool fused;              // dK/dV: one workgroup per key tile and kv head loops over the query heads (plain RMW)
    int64_t dq_blocks, dkv_blocks;
    bool ok;
};
// Upper bounds on tile counts: sum_g ceil(L_g / tile) <= total / tile + n_segments.
int64_t kv_tiles_most(const cf_attn_fwd_params &p) { return (int64_t)p.n_kv_tokens / (p.head_dim == 64 ? DkvShape<64>::BKV : BKV) + p.n_segments; }
int64_t q_tiles_most(const cf_attn_fwd_params &p) { return p.q_tiles ? (int64_t)p.n_q_tiles : (int64_t)p.n_tokens / BM + p.n_segments; }

BwdShape bwd_shape(const cf_attn_fwd_params &p, const BwdWorkspace &ws)
{
    BwdShape g;
    const int64_t kv_tiles = kv_tiles_most(p);
    // Fusing the heads of a group into one workgroup needs enough key tiles to fill 256 CUs several times.  At D = 64 dK/dV rows
    // always have one writer (and no work list).
    g.fused = kv_tiles * p.n_kv_heads >= 4096 || (p.flags & CF_FLAG_DKV_SINGLE_WRITER) || p.head_dim == 64;
    g.dq_blocks = q_tiles_most(p) * p.n_q_heads;
    g.dkv_blocks = (g.fused ? kv_tiles : ws.worklist_items) * p.n_kv_heads;
    g.ok = g.dkv_blocks <= 0x7fffffffLL && g.dq_blocks < 0x7fffffffLL && ws.worklist_items <= 0x7fffffffLL;
    return g;
}

template <int D>
hipError_t launch_dkv(const cf_attn_bwd_params &b, const BwdWorkspace &ws, const BwdShape &g, const ProfileHook &hook, hipStream_t s)
{
    if (hook.start) (void)hipEventRecord(hook.start, s);
    if (g.fused) mfma_dkv_kernel<D, true><<<dim3((unsigned)g.dkv_blocks), 256, 0, s>>>(b, ws.delta, nullptr);
    else if constexpr (D == 128) mfma_dkv_kernel<D, false><<<dim3((unsigned)g.dkv_blocks), 256, 0, s>>>(b, ws.delta, ws.worklist);
    const hipError_t e = hipGetLastError();
    if (hook.stop) (void)hipEventRecord(hook.stop, s);
    return e;
}

template <int D>
hipError_t run_bwd(const cf_attn_bwd_params &b, const BwdWorkspace &ws, hipStream_t s)
{
    const BwdShape g = bwd_shape(b.f, ws);
    if (!g.ok) return hipErrorInvalidConfiguration;
    // dQ first: it also produces delta, which the dK/dV kernel reads; its first workgroup builds the dK/dV work list
    // where one is needed.
    int *wl = g.fused ? nullptr : ws.worklist;
    const dim3 dq_grid((unsigned)(g.dq_blocks + (wl ? 1 : 0)));
    if (D == 64 || wide_mfma(b.f)) mfma_dq_kernel<D, 32><<<dq_grid, 256, 0, s>>>(b, ws.delta, wl, (int)ws.worklist_items);
    else if constexpr (D == 128) mfma_dq_kernel<D, 16><<<dq_grid, 256, 0, s>>>(b, ws.delta, wl, (int)ws.worklist_items);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_dkv<D>(b, ws, g, take_profile_hook(), s);
}

// Adds a chunk's part to a batch launch.
bool append(BwdBatch &q, const cf_attn_bwd_params &b, const BwdWorkspace &ws, const BwdShape &g, int64_t blocks)
{
    const int i = q.blocks.n;
    if (!q.blocks.append(blocks)) return false;
    q.capacity[i] = (int)ws.worklist_items;
    q.delta[i] = ws.delta;
    q.wl[i] = g.fused ? nullptr : ws.worklist;
    q.wide = (i == 0 ? 0 : q.wide) | (unsigned)wide_mfma(b.f) << i;
    q.b[i] = b;
    return true;
}

// How a chunk's dK/dV goes out.  Calls that add to the same rows do so in the order of the calls where each of them adds to a row once.
//   kList   a list that cuts key tiles into several items, which meet in atomic adds in any order; the lists of several slices then go
//           together, in any order too: a step of 28 / 4 heads, 4 slices of 512 tokens and 2 packed chunks 302 -> 234 us, 4 slices
//           of 1024 and 3 packed chunks 720 -> 580 (slices of 8192: no change, their launches end evenly)
//   kChain  one writer per row (D = 64), or a list of one item to a key tile: the slices of a sequence go from one to the next in the
//           workgroup of a key tile.  32 / 32 heads, 4000 tokens in slices of 512 and 2 packed chunks: 774 us a step, 1040 with a launch per
//           slice (lists in any order: 869); 8 / 8 heads, 20000 tokens in slices of 1000: 3933, 4600 (3810)
//   kAlone  a launch of its own, in order: one writer per row by the flag or for many key tiles; and lists of one item to a key tile whose
//           launches end evenly (32 / 32 heads, 16000 tokens in slices of 2000, up to 240 pairs a slot: 8.98 ms a step, as a chain 9.16)
enum DkvKind { kAlone, kList, kChain };
constexpr float kChainMost = 96;      // pairs a slot
// Of a call with a work list.  Are the key tiles that all its query tiles see cut into several items, in a launch of its own?
// (Several segments: their lengths are not known here; such a call shares rows with no other in a launch.)
DkvKind kind_of_list(const cf_attn_fwd_params &p, const BwdWorkspace &ws)
{
    if (p.n_segments > 1) return kList;
    const int64_t prefix = p.n_kv_tokens - p.n_tokens, q_tiles = ((int64_t)p.n_tokens + BQ - 1) / BQ;
    // key tiles up to the one with the first own row are seen by all query tiles, each one behind by 128 / 64 fewer
    const int64_t whole = prefix / BKV + 1, first = whole * BKV - prefix, rest = first < p.n_tokens ? (p.n_tokens - first + BKV - 1) / BKV : 0;
    static_assert(BKV == 2 * BQ, "the sum of the rest");
    const int64_t total = whole * q_tiles + rest * (q_tiles - first / BQ) - rest * (rest - 1);
    const int G = p.n_q_heads / p.n_kv_heads;
    const ListCuts cuts((int)std::min<int64_t>(total, 0x7fffffff), (int)(whole + rest), p.n_q_heads, kSlots);
    bool heads;
    if (cuts.items((int)q_tiles, G, true, heads) > 1 && (ws.worklist_items >= dkv_items_most(p) || cuts.items((int)q_tiles, G, false, heads) > 1)) return kList;
    return cuts.average <= kChainMost ? kChain : kAlone;
}
// Slices whose lists may add to the rows that they share in any order: all of these lie before the longer one's own rows, where its
// key tiles are cut.
bool any_order(const cf_attn_bwd_params &a, const cf_attn_bwd_params &c)
{
    const cf_attn_fwd_params &l = a.f.n_kv_tokens > c.f.n_kv_tokens ? a.f : c.f, &s = &l == &a.f ? c.f : a.f;
    return same_key_rows(a, c) && s.n_kv_tokens <= l.n_kv_tokens - l.n_tokens;
}

template <int D>
hipError_t run_bwd_batch(const BwdBatchChunk *chunks, int n, hipStream_t s)
{
    BwdShape g[CF_BWD_BATCH_MAX];
    int order[CF_BWD_BATCH_MAX], dq_order[CF_BWD_BATCH_MAX], slots[CF_BWD_BATCH_MAX];
    int64_t tokens[CF_BWD_BATCH_MAX] = {};           // of the dK/dV launch that a chunk goes into (index: its first chunk)
    int first_of[CF_BWD_BATCH_MAX], together[CF_BWD_BATCH_MAX] = {};
    DkvKind kind[CF_BWD_BATCH_MAX];
    unsigned shares = 0;                             // bit c: chunk c adds to rows that another one adds to
    for (int c = 0; c < n; ++c)
        if (chunks[c].meets != 0) shares |= chunks[c].meets | 1u << c;
    for (int c = 0; c < n; ++c) {
        g[c] = bwd_shape(chunks[c].b->f, chunks[c].ws);
        if (!g[c].ok) return hipErrorInvalidConfiguration;
        kind[c] = D == 64 ? kChain : g[c].fused ? kAlone : shares >> c & 1 ? kind_of_list(chunks[c].b->f, chunks[c].ws) : kList;
        first_of[c] = c > 0 && kind[c] == kind[c - 1] && kind[c] != kAlone ? first_of[c - 1] : c;
        for (int a = first_of[c]; a < c; ++a)
            if ((chunks[c].meets >> a & 1) && !(kind[c] == kChain ? same_key_rows : any_order)(*chunks[a].b, *chunks[c].b)) first_of[c] = c;
        order[c] = dq_order[c] = c;
    }
    for (int c = 0; c < n; ++c) tokens[first_of[c]] += chunks[c].b->f.n_tokens, ++together[first_of[c]];
    for (int c = 0; D == 128 && c < n; ++c)          // (a chain needs no list, and has a workgroup for each key tile)
        if (kind[c] == kChain && together[first_of[c]] > 1)
            g[c].fused = true, g[c].dkv_blocks = kv_tiles_most(chunks[c].b->f) * chunks[c].b->f.n_kv_heads;
    // dK/dV: heaviest first (the items of a list have no chains to speak of: by longest chain 28 / 4 heads, four packed chunks of 2048
    // tokens take 214 us, 208 so)
    std::stable_sort(order, order + n, [&](int x, int y) { return work_of(chunks[x].b->f) > work_of(chunks[y].b->f); });
    std::stable_sort(dq_order, dq_order + n, [&](int x, int y) { return starts_before(chunks[x].b->f, chunks[y].b->f); });
    for (int i = 0; i < n; ++i) {
        const int c = order[i];
        // Lists follow each other in a shared launch: the longest items of a late one start late and have to end with what is
        // left, so that a chunk's share of the slots is taken of the chunks from it on.
        const int64_t own = chunks[c].b->f.n_tokens;
        slots[c] = (int)max((int64_t)1, min((int64_t)kSlots - (together[first_of[c]] > 1), kSlots * own / tokens[first_of[c]]));
        tokens[first_of[c]] -= own;
    }
    BwdBatch q;
    q.blocks.clear();
    for (int i = 0; i < n; ++i) {
        const int c = dq_order[i];
        q.slots[i] = slots[c];
        if (!append(q, *chunks[c].b, chunks[c].ws, g[c], g[c].dq_blocks)) return hipErrorInvalidConfiguration;
    }
    const dim3 dq_grid((unsigned)(q.blocks.end + n));
    if (D == 64 || q.wide == (1u << n) - 1) mfma_dq_batch_kernel<D, 32><<<dq_grid, 256, 0, s>>>(q);
    else if constexpr (D == 128) {
        if (q.wide == 0) mfma_dq_batch_kernel<D, 16><<<dq_grid, 256, 0, s>>>(q);
        else mfma_dq_batch_kernel<D, 0><<<dq_grid, 256, 0, s>>>(q);
    }
    hipError_t e = hipGetLastError();
    for (int first = 0, end; first < n && e == hipSuccess; first = end) {
        for (end = first + 1; end < n && first_of[end] == first;) ++end;
        if (end == first + 1) {
            e = launch_dkv<D>(*chunks[first].b, chunks[first].ws, g[first], ProfileHook(), s);
            continue;
        }
        q.blocks.clear();
        if (kind[first] == kChain) {
            const CallChains<CF_BWD_BATCH_MAX> chain(end - first, [&](int c) -> const cf_attn_bwd_params & { return *chunks[first + c].b; });
            int place[CF_BWD_BATCH_MAX];
            for (int i = 0; i < end - first; ++i) place[chain.order[i]] = i;
            for (int i = 0; i < end - first; ++i) {
                const int c = chain.order[i];
                int64_t blocks = 0;                  // a chain's key tiles go with its first call: as many as its longest one has
                for (int a = c; chain.head[c] == c && a >= 0; a = chain.next[a]) blocks = std::max(blocks, g[first + a].dkv_blocks);
                if (!append(q, *chunks[first + c].b, chunks[first + c].ws, g[first + c], blocks)) return hipErrorInvalidConfiguration;
                q.next[i] = chain.next[c] < 0 ? -1 : place[chain.next[c]];
            }
        } else {
            for (int i = 0; i < n; ++i) {
                const int c = order[i];
                if (first_of[c] == first && !append(q, *chunks[c].b, chunks[c].ws, g[c], g[c].dkv_blocks)) return hipErrorInvalidConfiguration;
            }
        }
        const dim3 grid((unsigned)q.blocks.end);
        if (kind[first] == kChain) mfma_dkv_batch_kernel<D, true><<<grid, 256, 0, s>>>(q);
        else if constexpr (D == 128) mfma_dkv_batch_kernel<D, false><<<grid, 256, 0, s>>>(q);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

int64_t mfma_bwd_blocks(const cf_attn_fwd_params &p)
{
    const int64_t items = p.head_dim == 64 ? 0 : dkv_items_most(p);
    return std::max(q_tiles_most(p) * p.n_q_heads + 1, std::max(kv_tiles_most(p), items) * p.n_kv_heads);
}

int64_t dkv_worklist_least(const cf_attn_fwd_params &p) { return key_tiles_most(p) * (p.n_q_heads / p.n_kv_heads); }
int64_t dkv_worklist_capacity(const cf_attn_fwd_params &p) { return dkv_items_most(p); }

hipError_t launch_mfma_bwd(const cf_attn_bwd_params &b, const BwdWorkspace &ws, hipStream_t s)
{
    return b.f.head_dim == 64 ? run_bwd<64>(b, ws, s) : run_bwd<128>(b, ws, s);
}

hipError_t launch_mfma_bwd_batch(const BwdBatchChunk *chunks, int n, hipStream_t s)
{
    if (n < 1 || n > CF_BWD_BATCH_MAX) return hipErrorInvalidValue;
    return chunks[0].b->f.head_dim == 64 ? run_bwd_batch<64>(chunks, n, s) : run_bwd_batch<128>(chunks, n, s);
}

}  // namespace cf
