// C ABI of the device entry points: argument checks, workspace carving, kernel selection.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <vector>

#include "common.h"
#include "kernels.h"

namespace {

constexpr int kKnownFlags = CF_FLAG_SCALAR_KERNELS | CF_FLAG_DKV_SINGLE_WRITER;

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

int check_fwd(const cf_attn_fwd_params *p, const char *who, bool sizes_only)
{
    if (!p) return cf::fail(CF_EINVAL, "%s: params is NULL", who);
    if (p->dtype != CF_BF16 && p->dtype != CF_FP32)
        return cf::fail(CF_EUNSUPPORTED, "%s: dtype %d not supported", who, p->dtype);
    if (p->head_dim != 64 && p->head_dim != 128)
        return cf::fail(CF_EUNSUPPORTED, "%s: head_dim %d not supported (64 or 128)", who, p->head_dim);
    if (p->n_q_heads < 1 || p->n_kv_heads < 1 || p->n_q_heads % p->n_kv_heads != 0)
        return cf::fail(CF_EINVAL, "%s: n_q_heads %d must be a positive multiple of n_kv_heads %d", who,
                        p->n_q_heads, p->n_kv_heads);
    if (p->n_q_heads > 65535) return cf::fail(CF_EINVAL, "%s: n_q_heads %d > 65535", who, p->n_q_heads);
    if (p->n_tokens < 1 || p->n_segments < 1 || p->n_kv_tokens < p->n_tokens)
        return cf::fail(CF_EINVAL, "%s: need n_tokens >= 1, n_segments >= 1, n_kv_tokens >= n_tokens (got %d, %d, %d)",
                        who, p->n_tokens, p->n_segments, p->n_kv_tokens);
    if (p->n_segments > p->n_tokens)
        return cf::fail(CF_EINVAL, "%s: n_segments %d > n_tokens %d (empty segments are not allowed)", who,
                        p->n_segments, p->n_tokens);
    if (sizes_only) return CF_OK;
    if (p->flags & ~kKnownFlags) return cf::fail(CF_EINVAL, "%s: unknown flags 0x%x", who, p->flags);
    if (!p->cu_seqlens_q || !p->cu_seqlens_k || !p->q || !p->k || !p->v || !p->o || !p->lse)
        return cf::fail(CF_EINVAL, "%s: NULL device pointer", who);
    if (!(p->softmax_scale == p->softmax_scale))
        return cf::fail(CF_EINVAL, "%s: softmax_scale is NaN", who);
    const int64_t vec = p->dtype == CF_BF16 ? 8 : 4;  // elements per 16-byte access
    const int64_t D = p->head_dim;
    const int64_t strides[] = {p->q_stride_tok, p->q_stride_head, p->kv_stride_tok, p->kv_stride_head,
                               p->o_stride_tok, p->o_stride_head};
    for (int64_t s : strides)
        if (s < D || s % vec != 0)
            return cf::fail(CF_EINVAL, "%s: stride %lld must be >= head_dim and a multiple of %lld elements", who,
                            (long long)s, (long long)vec);
    if (!aligned(p->q, 16) || !aligned(p->k, 16) || !aligned(p->v, 16) || !aligned(p->o, 16) ||
        !aligned(p->lse, 4) || !aligned(p->cu_seqlens_q, 4) || !aligned(p->cu_seqlens_k, 4))
        return cf::fail(CF_EINVAL, "%s: q, k, v, o must be 16-byte aligned", who);
    // the optional tile table: between ceil(T / 128) and T / 128 + n_segments records of 32 bytes
    if ((p->q_tiles == nullptr) != (p->n_q_tiles == 0) || p->n_q_tiles < 0 || !aligned(p->q_tiles, 16))
        return cf::fail(CF_EINVAL, "%s: q_tiles / n_q_tiles = %d do not go together (NULL with 0, 16-byte aligned)", who,
                        p->n_q_tiles);
    if (p->q_tiles && (p->n_q_tiles < (p->n_tokens + 127) / 128 || p->n_q_tiles > p->n_tokens / 128 + p->n_segments))
        return cf::fail(CF_EINVAL, "%s: n_q_tiles = %d cannot be the tile count of %d tokens in %d segments", who,
                        p->n_q_tiles, p->n_tokens, p->n_segments);
    return CF_OK;
}

// Shapes the MFMA kernels cover (decides the workspace size, so it may only look at sizes, dtype, flags).
bool mfma_shape(const cf_attn_fwd_params &p)
{
    return p.dtype == CF_BF16 && !(p.flags & CF_FLAG_SCALAR_KERNELS);
}
// The matrix kernels address the rows of a block with 32-bit byte offsets: 63 rows x 2 bytes (bf16) and 31 rows x 4 bytes
// (fp32) of this many elements stay below 2^32.  Wider strides go to the scalar kernels.
constexpr int64_t kMostStride = 1 << 25;
bool narrow(const cf_attn_fwd_params &p) { return p.q_stride_tok < kMostStride && p.kv_stride_tok < kMostStride; }
// Their launches give every segment workgroups of its own: hundreds of thousands of segments can be more than one launch
// holds, and go to the scalar kernels (a row per wavefront).  (bf16 at head_dim 128 never had that way out.)
bool launchable_mfma(const cf_attn_fwd_params &p, bool backward)
{
    return p.head_dim == 128 || cf::mfma_launch_size(p, backward) <= cf::kMostWorkItems;
}
bool launchable_f32(const cf_attn_fwd_params &p, bool backward) { return cf::f32_launch_size(p, backward) <= cf::kMostWorkItems; }

// The MFMA kernels take the row maximum before scaling, which needs a positive scale.
bool use_mfma(const cf_attn_fwd_params &p) { return mfma_shape(p) && p.softmax_scale > 0.f && narrow(p) && launchable_mfma(p, false); }
bool use_mfma(const cf_attn_bwd_params &b) { return use_mfma(b.f) && b.do_stride_tok < kMostStride && launchable_mfma(b.f, true); }

// The fp32 matrix kernels: every fp32 shape, any scale.
bool use_f32(const cf_attn_fwd_params &p) { return p.dtype == CF_FP32 && !(p.flags & CF_FLAG_SCALAR_KERNELS) && narrow(p) && launchable_f32(p, false); }
bool use_f32(const cf_attn_bwd_params &b) { return use_f32(b.f) && b.do_stride_tok < kMostStride && launchable_f32(b.f, true); }

hipError_t fwd_one(const cf_attn_fwd_params &p, hipStream_t s)
{
    return use_mfma(p) ? cf::launch_mfma_fwd(p, s) : use_f32(p) ? cf::launch_f32_fwd(p, s) : cf::launch_simple_fwd(p, s);
}

int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

int64_t delta_bytes(const cf_attn_fwd_params &p) { return round_up((int64_t)p.n_q_heads * p.n_tokens * 4, 256); }
// counters (256 bytes) + 16-byte items; head_dim 64 has no work list
bool has_worklist(const cf_attn_fwd_params &p) { return mfma_shape(p) && p.head_dim == 128; }
int64_t worklist_bytes(const cf_attn_fwd_params &p) { return has_worklist(p) ? 256 + cf::dkv_worklist_capacity(p) * 16 : 0; }
// The least scratch a backward runs in: with room for the coarse list only, its work is cut less finely.
int64_t least_scratch(const cf_attn_fwd_params &p) { return delta_bytes(p) + (has_worklist(p) ? 256 + cf::dkv_worklist_least(p) * 16 : 0); }

int hip_fail(const char *who, hipError_t e)
{
    return cf::fail(CF_EHIP, "%s: %s", who, hipGetErrorString(e));
}

thread_local cf::ProfileHook g_hook;

}  // namespace

cf::ProfileHook cf::take_profile_hook()
{
    cf::ProfileHook h = g_hook;
    g_hook = cf::ProfileHook();
    return h;
}

extern "C" int cf_profile_next_call(void *start_event, void *stop_event)
{
    g_hook.start = start_event && stop_event ? static_cast<hipEvent_t>(start_event) : nullptr;
    g_hook.stop = start_event && stop_event ? static_cast<hipEvent_t>(stop_event) : nullptr;
    return CF_OK;
}

extern "C" int cf_attn_fwd(const cf_attn_fwd_params *p, void *hip_stream)
{
    if (int rc = check_fwd(p, "cf_attn_fwd", false)) return rc;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const hipError_t e = fwd_one(*p, s);
    return e == hipSuccess ? CF_OK : hip_fail("cf_attn_fwd", e);
}

extern "C" int64_t cf_attn_bwd_workspace_bytes(const cf_attn_fwd_params *p)
{
    if (int rc = check_fwd(p, "cf_attn_bwd_workspace_bytes", true)) return rc;
    if (p->flags & ~kKnownFlags)
        return cf::fail(CF_EINVAL, "cf_attn_bwd_workspace_bytes: unknown flags 0x%x", p->flags);
    return delta_bytes(*p) + worklist_bytes(*p);
}

namespace {

// Argument checks of one backward call apart from its scratch memory.
int check_bwd_tensors(const cf_attn_bwd_params *b, const char *who)
{
    if (!b) return cf::fail(CF_EINVAL, "%s: params is NULL", who);
    if (int rc = check_fwd(&b->f, who, false)) return rc;
    const cf_attn_fwd_params &p = b->f;
    if (!b->d_o || !b->d_q || !b->d_k || !b->d_v)
        return cf::fail(CF_EINVAL, "%s: NULL device pointer", who);
    const int64_t vec = p.dtype == CF_BF16 ? 8 : 4, D = p.head_dim;
    const int64_t strides[] = {b->do_stride_tok, b->do_stride_head, b->dq_stride_tok, b->dq_stride_head};
    for (int64_t s : strides)
        if (s < D || s % vec != 0)
            return cf::fail(CF_EINVAL, "%s: stride %lld must be >= head_dim and a multiple of %lld elements", who,
                            (long long)s, (long long)vec);
    if (b->dkv_stride_tok < D || b->dkv_stride_head < D || b->dkv_stride_tok % 4 || b->dkv_stride_head % 4)
        return cf::fail(CF_EINVAL, "%s: d_k/d_v strides must be >= head_dim and multiples of 4 elements", who);
    if (!aligned(b->d_o, 16) || !aligned(b->d_q, 16) || !aligned(b->d_k, 16) || !aligned(b->d_v, 16))
        return cf::fail(CF_EINVAL, "%s: d_o, d_q, d_k, d_v must be 16-byte aligned", who);
    return CF_OK;
}

// Lays the backward's scratch (delta, then the dK/dV work list) out in `bytes` bytes of device memory at `base`.
int carve_workspace(const cf_attn_fwd_params &p, void *base, int64_t bytes, const char *who, const char *what,
                    cf::BwdWorkspace *ws)
{
    if (!base || !aligned(base, 256)) return cf::fail(CF_EINVAL, "%s: %s must be non-NULL and 256-byte aligned", who, what);
    const int64_t need = least_scratch(p);
    if (bytes < need)
        return cf::fail(CF_EINVAL, "%s: %s has %lld bytes, %lld needed", who, what, (long long)bytes, (long long)need);
    ws->delta = static_cast<float *>(base);
    ws->worklist = has_worklist(p) ? reinterpret_cast<int *>(static_cast<char *>(base) + delta_bytes(p)) : nullptr;
    ws->worklist_items = has_worklist(p) ? std::min(cf::dkv_worklist_capacity(p), (bytes - delta_bytes(p) - 256) / 16) : 0;
    return CF_OK;
}

// Argument checks of one backward call; on success fills the scratch layout inside the caller's workspace.
int check_bwd(const cf_attn_bwd_params *b, const char *who, cf::BwdWorkspace *ws)
{
    if (int rc = check_bwd_tensors(b, who)) return rc;
    return carve_workspace(b->f, b->workspace, b->workspace_bytes, who, "workspace", ws);
}

int bwd_one(const cf_attn_bwd_params *b, const cf::BwdWorkspace &ws, hipStream_t s, const char *who)
{
    hipError_t e = hipSuccess;
    if (use_mfma(*b)) {
        e = cf::launch_mfma_bwd(*b, ws, s);          // its dQ kernel forms delta itself
    } else if (use_f32(*b)) {
        e = cf::launch_f32_bwd(*b, s);               // so does every workgroup of this one
    } else {
        e = cf::launch_delta(*b, ws, s);
        if (e != hipSuccess) return hip_fail(who, e);
        e = cf::launch_simple_bwd(*b, ws, s);
    }
    return e == hipSuccess ? CF_OK : hip_fail(who, e);
}

// ---- several calls at once --------------------------------------------------------------------------------------
// Small chunks leave most of the chip idle and large ones end with a partly filled wave of workgroups: calls
// of one kind that do not touch each other's results go out as ONE launch (backward: one per kernel).  A step of 16
// chunks of 512 tokens, 28 / 4 heads: 769 us in 48 launches, 218 us in 3; 16 chunks of 8192 tokens: 9.43 -> 8.95 ms.
constexpr int kWindow = 64;      // calls looked at together

enum Path { kScalar, kMfma, kF32 };
// A checked call: f of a forward (b NULL) or of a backward, whose scratch ws is; and what a list is ordered by, looked up once a call (host
// time of a step's lists, 16 packed chunks: 14.7 -> 14.2 us, 13 small fp32 calls: 7.4 -> 7.2).
struct Call {
    const cf_attn_fwd_params *f;
    const cf_attn_bwd_params *b;
    cf::BwdWorkspace ws;
    Path path;
    uint64_t kernel;             // the same in calls that can share launches; 0: it shares none
    int64_t size;                // work-items of its largest launch

    Call() = default;
    explicit Call(const cf_attn_fwd_params *fwd)
        : f(fwd), b(nullptr), ws(), path(use_mfma(*f) ? kMfma : use_f32(*f) ? kF32 : kScalar), kernel(kernel_of()), size(size_of()) {}
    Call(const cf_attn_bwd_params *bwd, const cf::BwdWorkspace &scratch)
        : f(&bwd->f), b(bwd), ws(scratch), path(use_mfma(*b) ? kMfma : use_f32(*b) ? kF32 : kScalar), kernel(kernel_of()), size(size_of()) {}

private:
    uint64_t kernel_of() const       // (at most 65535 heads)
    {
        return path == kScalar ? 0 : (uint64_t)path << 48 | (uint64_t)(b != nullptr) << 40 | (uint64_t)f->head_dim << 32 | (uint64_t)f->n_q_heads << 16 | (uint64_t)f->n_kv_heads;
    }
    int64_t size_of() const
    {
        return path == kMfma ? cf::mfma_launch_size(*f, b != nullptr) : path == kF32 ? cf::f32_launch_size(*f, b != nullptr) : cf::simple_launch_size(*f, b != nullptr);
    }
};
bool same_kernel(const Call &a, const Call &c) { return a.kernel != 0 && a.kernel == c.kernel; }

// Memory that a call touches, as address ranges (of a strided tensor: from its first to its last element).
struct Range {
    uintptr_t begin, end;
    bool meets(const Range &o) const { return begin < o.end && o.begin < end; }
};
struct Touched {
    Range reads[6], writes[2], adds[2];
    int n_reads, n_adds;
};
Range tensor_range(const void *base, int64_t rows, int64_t stride_tok, int64_t heads, int64_t stride_head, int64_t D, int64_t elem)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(base);
    return {a, a + (uintptr_t)(((rows - 1) * stride_tok + (heads - 1) * stride_head + D) * elem)};
}
Touched touched(const Call &c)
{
    const cf_attn_fwd_params &p = *c.f;
    const int64_t D = p.head_dim, elem = p.dtype == CF_BF16 ? 2 : 4, T = p.n_tokens, H = p.n_q_heads;
    const Range o = tensor_range(p.o, T, p.o_stride_tok, H, p.o_stride_head, D, elem), lse = tensor_range(p.lse, H, T, 1, 0, T, 4);
    Touched t;
    t.reads[0] = tensor_range(p.q, T, p.q_stride_tok, H, p.q_stride_head, D, elem);
    t.reads[1] = tensor_range(p.k, p.n_kv_tokens, p.kv_stride_tok, p.n_kv_heads, p.kv_stride_head, D, elem);
    t.reads[2] = tensor_range(p.v, p.n_kv_tokens, p.kv_stride_tok, p.n_kv_heads, p.kv_stride_head, D, elem);
    t.n_reads = c.b ? 6 : 3;
    t.n_adds = c.b ? 2 : 0;
    if (!c.b) {
        t.writes[0] = o, t.writes[1] = lse;
        return t;
    }
    const cf_attn_bwd_params &b = *c.b;
    t.reads[3] = o, t.reads[4] = lse;
    t.reads[5] = tensor_range(b.d_o, T, b.do_stride_tok, H, b.do_stride_head, D, elem);
    t.writes[0] = tensor_range(b.d_q, T, b.dq_stride_tok, H, b.dq_stride_head, D, elem);
    t.writes[1] = {reinterpret_cast<uintptr_t>(b.workspace), reinterpret_cast<uintptr_t>(b.workspace) + (uintptr_t)b.workspace_bytes};
    t.adds[0] = tensor_range(b.d_k, p.n_kv_tokens, b.dkv_stride_tok, p.n_kv_heads, b.dkv_stride_head, D, 4);
    t.adds[1] = tensor_range(b.d_v, p.n_kv_tokens, b.dkv_stride_tok, p.n_kv_heads, b.dkv_stride_head, D, 4);
    return t;
}
bool any_meet(const Range *a, int na, const Range *c, int nc)
{
    for (int i = 0; i < na; ++i)
        for (int j = 0; j < nc; ++j)
            if (a[i].meets(c[j])) return true;
    return false;
}
bool adds_meet(const Touched &a, const Touched &c) { return any_meet(a.adds, a.n_adds, c.adds, c.n_adds); }
// The fp32 kernel takes both calls in one launch: one writer per gradient row goes from slice to slice.
bool chains(const Call &a, const Touched &ta, const Call &c, const Touched &tc) { return !adds_meet(ta, tc) || cf::same_key_rows(*a.b, *c.b); }
// Apart from gradients that both add to, neither reads or writes what the other writes.
bool independent(const Touched &a, const Touched &c)
{
    return !any_meet(a.writes, 2, c.reads, c.n_reads) && !any_meet(a.reads, a.n_reads, c.writes, 2) && !any_meet(a.writes, 2, c.writes, 2) &&
           !any_meet(a.adds, a.n_adds, c.reads, c.n_reads) && !any_meet(a.reads, a.n_reads, c.adds, c.n_adds) &&
           !any_meet(a.adds, a.n_adds, c.writes, 2) && !any_meet(a.writes, 2, c.adds, c.n_adds);
}

int launch_together(const Call *calls, const Touched *t, int n, hipStream_t s, const char *who)
{
    static_assert(cf::CF_BWD_BATCH_MAX <= cf::CF_FWD_BATCH_MAX, "sizes the arrays below");
    hipError_t e;
    if (n == 1) {
        if (calls[0].b) return bwd_one(calls[0].b, calls[0].ws, s, who);
        e = fwd_one(*calls[0].f, s);
        return e == hipSuccess ? CF_OK : hip_fail(who, e);
    }
    if (calls[0].b && calls[0].path == kMfma) {
        cf::BwdBatchChunk chunks[cf::CF_BWD_BATCH_MAX];
        for (int c = 0; c < n; ++c) {
            chunks[c] = {calls[c].b, calls[c].ws, 0};
            for (int a = 0; a < c; ++a) chunks[c].meets |= (unsigned)adds_meet(t[a], t[c]) << a;
        }
        e = cf::launch_mfma_bwd_batch(chunks, n, s);
        return e == hipSuccess ? CF_OK : hip_fail(who, e);
    }
    if (calls[0].b) {
        const cf_attn_bwd_params *bwd[cf::CF_BWD_BATCH_MAX];
        for (int c = 0; c < n; ++c) bwd[c] = calls[c].b;
        e = cf::launch_f32_bwd_batch(bwd, n, s);
        return e == hipSuccess ? CF_OK : hip_fail(who, e);
    }
    const cf_attn_fwd_params *fwd[cf::CF_FWD_BATCH_MAX];
    for (int i = 0; i < n; ++i) fwd[i] = calls[i].f;
    std::stable_sort(fwd, fwd + n, [](const cf_attn_fwd_params *x, const cf_attn_fwd_params *y) { return cf::starts_before(*x, *y); });
    e = calls[0].path == kMfma ? cf::launch_mfma_fwd_batch(fwd, n, s) : cf::launch_f32_fwd_batch(fwd, n, s);
    return e == hipSuccess ? CF_OK : hip_fail(who, e);
}

// Brings calls of one kernel together: a call moves forward, behind the last one of the run that it joins, past calls of other kernels that
// it has nothing to do with (neither reads or writes what the other writes, no common gradient rows).  order: of t, from the first call to
// the last; calls of one kernel keep theirs.  Algorithm 2's second half asks for forward and backward in turns (one kept chunk: a slice's
// forward again, its backward, the slice before it, ...): launches of one slice each, which fill the chip in part.  Steps, us: a sequence
// of 32768 in slices of 2048 and a packed chunk, 28 / 4 heads, one kept chunk: 35590 -> 33920 (host time of the list 145-210 -> 24: its 34
// launches become 4); 9000 in slices of 1024 and 2 packed chunks, two kept: 3524 -> 2605; 8000 in slices of 512 and 2 packed chunks, 8 / 2
// heads, one kept: 3737 -> 1071.
void bring_together(const Call *calls, const Touched *t, int n, int *order)
{
    bool placed[kWindow] = {};
    for (int at = 0, first = 0; at < n;) {
        while (placed[first]) ++first;
        order[at++] = first;
        placed[first] = true;
        for (int j = first + 1; j < n; ++j) {
            if (placed[j] || !same_kernel(calls[first], calls[j])) continue;
            bool free = true;                        // of all that stay behind it and were before it
            for (int a = first + 1; a < j && free; ++a) free = placed[a] || (independent(t[a], t[j]) && !adds_meet(t[a], t[j]));
            if (!free) break;
            order[at++] = j;
            placed[j] = true;
        }
    }
}

// Launches n <= kWindow checked calls, in an order that gives the results of theirs.
int launch_calls(const Call *in, int n, hipStream_t s, const char *who)
{
    Touched touches[kWindow], t[kWindow];
    Call calls[kWindow];
    int order[kWindow];
    bool keep = true;                                // the order: one kernel, or a call that may be refused by its launch
    for (int i = 0; i < n; ++i) {
        touches[i] = touched(in[i]);
        order[i] = i;
        keep = keep && same_kernel(in[0], in[i]);
    }
    for (int i = 0; i < n && !keep; ++i) keep = in[i].size > cf::kMostWorkItems;
    if (!keep) bring_together(in, touches, n, order);
    for (int i = 0; i < n; ++i) calls[i] = in[order[i]], t[i] = touches[order[i]];
    for (int i = 0; i < n;) {
        int end = i + 1;
        while (end < n && same_kernel(calls[i], calls[end])) ++end;
        // a run that needs several launches is split evenly
        const int most = calls[i].b ? cf::CF_BWD_BATCH_MAX : cf::CF_FWD_BATCH_MAX;
        const int launches = (end - i + most - 1) / most, size = (end - i + launches - 1) / launches;
        while (i < end) {
            int64_t work_items = calls[i].size;
            int j = i + 1;
            for (; j < end && j - i < size; ++j) {
                work_items += calls[j].size;
                if (work_items > cf::kMostWorkItems) break;
                bool apart = true;
                for (int a = i; a < j && apart; ++a)
                    apart = independent(t[a], t[j]) && (!calls[j].b || calls[j].path != kF32 || chains(calls[a], t[a], calls[j], t[j]));
                if (!apart) break;
            }
            if (int rc = launch_together(calls + i, t + i, j - i, s, who)) return rc;
            i = j;
        }
    }
    return CF_OK;
}

}  // namespace

extern "C" int cf_attn_bwd(const cf_attn_bwd_params *b, void *hip_stream)
{
    cf::BwdWorkspace ws;
    if (int rc = check_bwd(b, "cf_attn_bwd", &ws)) return rc;
    return bwd_one(b, ws, static_cast<hipStream_t>(hip_stream), "cf_attn_bwd");
}

// ---- the backward for callers that cannot allocate -------------------------------------------------------------
// The scratch of cf_attn_bwd_static: one array per GPU, part of the loaded code object, alive until the process
// ends.  Host code never uses the array's name as an address: the device address is looked up once per device
// (hipGetSymbolAddress with that device current) and kept in g_static_scratch.
static __device__ __align__(256) unsigned char scratch[CF_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void *> g_static_scratch[kMaxDevices];

// Device address of `scratch` on the current device.
int static_scratch(const char *who, void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(who, e);
    if (dev < 0 || dev >= kMaxDevices) return cf::fail(CF_EUNSUPPORTED, "%s: device ordinal %d out of range", who, dev);
    void *ptr = g_static_scratch[dev].load(std::memory_order_acquire);
    if (!ptr) {
        // (two threads racing here both get the same address from the runtime)
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(who, e);
        if (!ptr) return cf::fail(CF_EHIP, "%s: hipGetSymbolAddress returned a NULL address", who);
        g_static_scratch[dev].store(ptr, std::memory_order_release);
    }
    *out = ptr;
    return CF_OK;
}
}  // namespace

extern "C" int cf_attn_bwd_static(const cf_attn_bwd_params *b, void *hip_stream)
{
    const char *who = "cf_attn_bwd_static";
    if (int rc = check_bwd_tensors(b, who)) return rc;
    // the size check comes before any HIP call: an oversized chunk is refused on any host
    const int64_t need = least_scratch(b->f);
    if (need > (int64_t)CF_STATIC_SCRATCH_BYTES)
        return cf::fail(CF_EINVAL, "%s: this chunk needs %lld bytes of scratch, the static buffer holds %lld "
                        "(use cf_attn_bwd with a workspace)", who, (long long)need, (long long)CF_STATIC_SCRATCH_BYTES);
    void *base = nullptr;
    if (int rc = static_scratch(who, &base)) return rc;
    cf::BwdWorkspace ws;
    if (int rc = carve_workspace(b->f, base, CF_STATIC_SCRATCH_BYTES, who, "static scratch", &ws)) return rc;
    return bwd_one(b, ws, static_cast<hipStream_t>(hip_stream), who);
}

extern "C" int cf_attn_fwd_batch(const cf_attn_fwd_params *params, int32_t n, void *hip_stream)
{
    const char *who = "cf_attn_fwd_batch";
    (void)cf::take_profile_hook();      // the hook times single-chunk calls only: an armed one ends here, unused
    if (n < 0 || (n > 0 && !params)) return cf::fail(CF_EINVAL, "%s: bad argument", who);
    for (int32_t i = 0; i < n; ++i)
        if (int rc = check_fwd(&params[i], who, false)) return rc;
    Call calls[kWindow];
    for (int32_t i = 0; i < n; i += kWindow) {
        const int m = std::min(n - i, kWindow);
        for (int a = 0; a < m; ++a) calls[a] = Call(&params[i + a]);
        if (int rc = launch_calls(calls, m, static_cast<hipStream_t>(hip_stream), who)) return rc;
    }
    return CF_OK;
}

extern "C" int cf_attn_bwd_batch(const cf_attn_bwd_params *params, int32_t n, void *hip_stream)
{
    const char *who = "cf_attn_bwd_batch";
    (void)cf::take_profile_hook();      // the hook times single-chunk calls only: an armed one ends here, unused
    if (n < 0 || (n > 0 && !params)) return cf::fail(CF_EINVAL, "%s: bad argument", who);
    std::vector<cf::BwdWorkspace> ws;
    try {
        ws.resize((size_t)n);
    } catch (const std::bad_alloc &) {
        return cf::fail(CF_ENOMEM, "%s: out of host memory", who);
    }
    for (int32_t i = 0; i < n; ++i)
        if (int rc = check_bwd(&params[i], who, &ws[i])) return rc;
    // the chunks of one call run interleaved: their workspaces must not overlap
    for (int32_t i = 0; i < n; ++i)
        for (int32_t j = i + 1; j < n; ++j) {
            const char *a = static_cast<const char *>(params[i].workspace), *b = static_cast<const char *>(params[j].workspace);
            if (a < b + params[j].workspace_bytes && b < a + params[i].workspace_bytes)
                return cf::fail(CF_EINVAL, "%s: chunks %d and %d share workspace memory", who, i, j);
        }
    Call calls[kWindow];
    for (int32_t i = 0; i < n; i += kWindow) {
        const int m = std::min(n - i, kWindow);
        for (int a = 0; a < m; ++a) calls[a] = Call(&params[i + a], ws[i + a]);
        if (int rc = launch_calls(calls, m, static_cast<hipStream_t>(hip_stream), who)) return rc;
    }
    return CF_OK;
}

extern "C" int cf_attn_calls(const cf_attn_call *calls, int64_t n, void *hip_stream)
{
    if (n < 0 || (n > 0 && !calls)) return cf::fail(CF_EINVAL, "cf_attn_calls: bad argument");
    Call window[kWindow];
    for (int64_t i = 0; i < n;) {
        int m = 0, bad = CF_OK;
        // (the profile hook is for one call: that call goes alone)
        for (const int most = g_hook.start ? 1 : kWindow; m < most && i + m < n; ++m) {
            const cf_attn_call &c = calls[i + m];
            if (c.backward) {
                const auto *b = static_cast<const cf_attn_bwd_params *>(c.params);
                cf::BwdWorkspace ws;
                bad = check_bwd(b, "cf_attn_bwd", &ws);
                if (!bad) window[m] = Call(b, ws);
            } else {
                const auto *f = static_cast<const cf_attn_fwd_params *>(c.params);
                bad = check_fwd(f, "cf_attn_fwd", false);
                if (!bad) window[m] = Call(f);
            }
            if (bad) break;
        }
        if (int rc = launch_calls(window, m, static_cast<hipStream_t>(hip_stream), "cf_attn_calls")) return rc;
        if (bad) return bad;
        i += m;
    }
    return CF_OK;
}
