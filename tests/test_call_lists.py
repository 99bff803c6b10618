"""What cf_attn_calls enqueues of a list, in which order, and what of it when a launch fails: the host code of csrc/api.hip over launchers
that only print (no GPU)."""
import os
import subprocess

import pytest

from paper_2503_02356_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")

PROGRAM = r"""
#include "api.hip"
#include <cstdarg>
#include <cstdio>

namespace {
int refused = -1;                // the call whose launch fails
char *buffer(long long i) { return reinterpret_cast<char *>((i + 1) << 40); }
const int32_t *bounds() { return reinterpret_cast<const int32_t *>(buffer(200)); }
int number(const cf_attn_fwd_params &p) { return (int)(p.cu_seqlens_q - bounds()); }      // (never read, so it tells the calls apart)
hipError_t launched(const char *kernel, const cf_attn_fwd_params *const *p, int n)
{
    for (int i = 0; i < n; ++i)
        if (number(*p[i]) == refused) return hipErrorInvalidConfiguration;
    std::printf("%s", kernel);
    for (int i = 0; i < n; ++i) std::printf(" %d", number(*p[i]));
    std::printf("\n");
    return hipSuccess;
}
hipError_t launched(const char *kernel, const cf_attn_fwd_params &p)
{
    const cf_attn_fwd_params *one = &p;
    return launched(kernel, &one, 1);
}
}  // namespace

namespace cf {
int fail(int code, const char *, ...) { return code; }
int64_t dkv_worklist_capacity(const cf_attn_fwd_params &) { return 1; }
int64_t dkv_worklist_least(const cf_attn_fwd_params &) { return 1; }
int64_t f32_launch_size(const cf_attn_fwd_params &p, bool) { return p.n_tokens; }
int64_t mfma_launch_size(const cf_attn_fwd_params &p, bool) { return p.n_tokens; }
hipError_t launch_f32_fwd(const cf_attn_fwd_params &p, hipStream_t) { return launched("fp32 forward", p); }
hipError_t launch_f32_bwd(const cf_attn_bwd_params &b, hipStream_t) { return launched("fp32 backward", b.f); }
hipError_t launch_simple_fwd(const cf_attn_fwd_params &p, hipStream_t) { return launched("scalar forward", p); }
hipError_t launch_simple_bwd(const cf_attn_bwd_params &b, const BwdWorkspace &, hipStream_t) { return launched("scalar backward", b.f); }
hipError_t launch_delta(const cf_attn_bwd_params &, const BwdWorkspace &, hipStream_t) { return hipSuccess; }
hipError_t launch_mfma_fwd(const cf_attn_fwd_params &p, hipStream_t) { return launched("bf16 forward", p); }
hipError_t launch_mfma_bwd(const cf_attn_bwd_params &b, const BwdWorkspace &, hipStream_t) { return launched("bf16 backward", b.f); }
hipError_t launch_f32_fwd_batch(const cf_attn_fwd_params *const *c, int n, hipStream_t) { return launched("fp32 forward", c, n); }
hipError_t launch_mfma_fwd_batch(const cf_attn_fwd_params *const *c, int n, hipStream_t) { return launched("bf16 forward", c, n); }
hipError_t launch_f32_bwd_batch(const cf_attn_bwd_params *const *c, int n, hipStream_t)
{
    const cf_attn_fwd_params *f[16];
    for (int i = 0; i < n; ++i) f[i] = &c[i]->f;
    return launched("fp32 backward", f, n);
}
hipError_t launch_mfma_bwd_batch(const BwdBatchChunk *c, int n, hipStream_t)
{
    const cf_attn_fwd_params *f[16];
    for (int i = 0; i < n; ++i) f[i] = &c[i].b->f;
    return launched("bf16 backward", f, n);
}
}  // namespace cf

// Arguments: the number of the call that its launch refuses (-1: none).  Calls from standard input, one a line: backward, data type, scalar
// kernels, query rows, segments, and the numbers of the buffers that it reads as Q, K / V and writes as O / LSE.
int main(int argc, char **argv)
{
    static cf_attn_bwd_params calls[64];
    cf_attn_call list[64];
    refused = argc > 1 ? std::atoi(argv[1]) : -1;
    int n = 0;
    for (long long backward, type, scalar, rows, segments, q, kv, out;
         n < 64 && std::scanf("%lld %lld %lld %lld %lld %lld %lld %lld", &backward, &type, &scalar, &rows, &segments, &q, &kv, &out) == 8; ++n) {
        cf_attn_bwd_params &b = calls[n];
        cf_attn_fwd_params &p = b.f;
        p.dtype = type ? CF_FP32 : CF_BF16, p.flags = scalar ? CF_FLAG_SCALAR_KERNELS : 0;
        p.n_q_heads = p.n_kv_heads = 1, p.head_dim = 64, p.softmax_scale = 1;
        p.n_tokens = p.n_kv_tokens = (int)rows, p.n_segments = (int)segments;
        p.q_stride_tok = p.q_stride_head = p.kv_stride_tok = p.kv_stride_head = p.o_stride_tok = p.o_stride_head = 64;
        p.cu_seqlens_q = p.cu_seqlens_k = bounds() + n;
        p.q = buffer(q), p.k = buffer(kv), p.v = buffer(kv) + (1LL << 39), p.o = buffer(out), p.lse = reinterpret_cast<float *>(buffer(out) + (1LL << 39));
        b.d_o = buffer(201);
        b.do_stride_tok = b.do_stride_head = b.dq_stride_tok = b.dq_stride_head = b.dkv_stride_tok = b.dkv_stride_head = 64;
        b.d_q = buffer(300 + n), b.workspace = buffer(400 + n), b.workspace_bytes = 1LL << 38;
        b.d_k = reinterpret_cast<float *>(buffer(500 + n)), b.d_v = reinterpret_cast<float *>(buffer(600 + n));
        list[n] = {backward ? static_cast<const void *>(&b) : &p, (int32_t)backward, 0};
    }
    std::printf("%d\n", cf_attn_calls(list, n, nullptr));
}
"""
FWD, BWD, BF16, FP32 = 0, 1, 0, 1


def call(backward, dtype=BF16, scalar=0, rows=100, segments=1, q=100, kv=101, out=0):
    return (backward, dtype, scalar, rows, segments, q, kv, out)


@pytest.fixture(scope="module")
def enqueued(tmp_path_factory):
    d = tmp_path_factory.mktemp("lists")
    (d / "lists.hip").write_text(PROGRAM)
    subprocess.run([build.HIPCC] + build.HIP_FLAGS + ["-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, str(d / "lists.hip"),
                    "-o", str(d / "lists")], check=True, stderr=subprocess.DEVNULL)

    def run(calls, refused=-1):
        text = "\n".join(" ".join(map(str, c)) for c in calls)
        lines = subprocess.run([str(d / "lists"), str(refused)], input=text, check=True, stdout=subprocess.PIPE, text=True).stdout.splitlines()
        launches = [(l.rstrip("0123456789 "), [int(x) for x in l[len(l.rstrip("0123456789 ")):].split()]) for l in lines[:-1]]
        return launches, int(lines[-1])
    return run


def test_calls_of_one_kernel_come_together(enqueued):
    turns = [call(kind, out=i // 2) for i in range(8) for kind in [(FWD, BWD)[i % 2]]]
    launches, rc = enqueued(turns)
    assert rc == 0 and [(k, sorted(c)) for k, c in launches] == [("bf16 forward", [0, 2, 4, 6]), ("bf16 backward", [1, 3, 5, 7])]
    mixed = [call(FWD, out=0), call(FWD, FP32, out=1), call(FWD, out=2), call(FWD, scalar=1, out=3), call(FWD, FP32, out=4)]
    launches, rc = enqueued(mixed)
    assert rc == 0 and [(k, sorted(c)) for k, c in launches] == [("bf16 forward", [0, 2]), ("fp32 forward", [1, 4]), ("scalar forward", [3])]


def test_no_call_passes_one_that_it_depends_on(enqueued):
    one_slot = [call(kind, out=0) for kind in (FWD, BWD, FWD, BWD)]
    assert enqueued(one_slot) == ([("bf16 forward", [0]), ("bf16 backward", [1]), ("bf16 forward", [2]), ("bf16 backward", [3])], 0)
    reads_the_first = [call(FWD, out=0), call(FWD, FP32, q=0, out=1), call(FWD, q=1, out=2)]
    assert [c for _, c in enqueued(reads_the_first)[0]] == [[0], [1], [2]]


def test_a_refused_call_ends_its_list(enqueued):
    """Refused by its arguments: the calls before it have been enqueued, those behind it have not."""
    calls = [call(FWD, out=0), call(FWD, FP32, out=1), call(FWD, rows=0), call(FWD, out=3)]
    assert enqueued(calls) == ([("bf16 forward", [0]), ("fp32 forward", [1])], -1)


@pytest.mark.parametrize("kind,rows,segments", [(FWD, 1 << 27, 1), (BWD, 1 << 27, 1), (BWD, 1 << 21, 1 << 21)])
def test_a_scalar_call_of_more_than_a_launch_holds_ends_its_list(enqueued, kind, rows, segments):
    """2^32 work-items in a row of workgroups, which the runtime refuses: 64 to a row of Q, or 4096 to a segment in the first kernel of the
    backward.  The call behind it, which the launch before it could take along, stays where it is."""
    calls = [call(FWD, out=0), call(kind, scalar=1, rows=rows, segments=segments, out=1), call(FWD, out=2)]
    assert enqueued(calls, refused=1) == ([("bf16 forward", [0])], -4)
    assert [c for _, c in enqueued(calls)[0]] == [[0], [1], [2]]
