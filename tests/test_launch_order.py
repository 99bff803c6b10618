"""The order in which the calls of a list start in the launches that they share (host code of csrc/kernels.h, compiled into a small program;
no GPU).  A launch ends with its longest chain, so the call that has it has to start first."""
import os
import subprocess

import pytest

from paper_2503_02356_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "kernels.h"
// calls from standard input, one a line: query rows, keys, segments, number of the gradient buffer (calls of one add to the same rows)
int main(int argc, char **argv)
{
    static cf_attn_bwd_params calls[16];
    static float gradients[64];
    int n = 0;
    for (long long rows, keys, segments, gradient; n < 16 && std::scanf("%lld %lld %lld %lld", &rows, &keys, &segments, &gradient) == 4; ++n) {
        calls[n].f.n_tokens = (int)rows, calls[n].f.n_kv_tokens = (int)keys, calls[n].f.n_segments = (int)segments;
        calls[n].d_k = gradients + 2 * gradient, calls[n].d_v = gradients + 2 * gradient + 1;
        calls[n].dkv_stride_tok = calls[n].dkv_stride_head = 64;
    }
    if (argc > 1 && std::strcmp(argv[1], "chains") == 0) {
        const cf::CallChains<16> chains(n, [&](int c) -> const cf_attn_bwd_params & { return calls[c]; });
        for (int i = 0; i < n; ++i) std::printf("%d ", chains.order[i]);
    } else {
        int order[16];
        for (int i = 0; i < n; ++i) order[i] = i;
        std::stable_sort(order, order + n, [&](int x, int y) { return cf::starts_before(calls[x].f, calls[y].f); });
        for (int i = 0; i < n; ++i) std::printf("%d ", order[i]);
    }
}
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text(PROGRAM)
    subprocess.run([build.HIPCC, "-O1", "-std=c++17", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-I", os.path.join(os.path.dirname(
        os.path.dirname(build.HIPCC)), "include"), "-D__HIP_PLATFORM_AMD__", "-x", "c++", str(d / "order.cpp"), "-o", str(d / "order")], check=True)

    def run(kind, calls):
        text = "\n".join(" ".join(map(str, c)) for c in calls)
        return [int(x) for x in subprocess.run([str(d / "order"), kind], input=text, check=True, stdout=subprocess.PIPE, text=True).stdout.split()]
    return run


def slices(n, rows, gradient):
    return [(rows, rows * (i + 1), 1, gradient) for i in range(n)]


def test_forward_and_dq_start_with_the_longest_chain_of_keys(order):
    late, packed, whole = (20, 620, 1, 0), (300, 300, 3, 1), (290, 290, 1, 2)
    assert order("rows", [packed, whole, late]) == [2, 0, 1]          # the late slice has the least work and the longest chain
    assert order("rows", [(4096, 4096, 20, 0), (904, 5000, 1, 1)]) == [1, 0]
    assert order("rows", [(300, 300, 30, 0), (300, 300, 3, 1), (300, 300, 10, 2)]) == [1, 2, 0]     # longer sequences first
    assert order("rows", [(100, 100, 1, 0), (100, 100, 1, 1)]) == [0, 1]                             # alike: as in the list


@pytest.mark.parametrize("n,rows", [(15, 500), (15, 256), (8, 1000), (3, 511), (2, 1300)])
def test_chains_start_by_the_rows_of_the_whole_chain(order, n, rows):
    """Slices whose rows are no multiple of 512: what counts is their sum, also where each is shorter than the step.  Beside the chain, a
    packed chunk of more work whose sequences are a step shorter than the chain."""
    total = n * rows
    tokens = 20 * total
    packed = (tokens, tokens, -(-4 * tokens // (total - 520)), 1)     # (the longest counts as four times the mean)
    assert order("chains", [packed] + slices(n, rows, 0)) == list(range(1, n + 1)) + [0]


def test_chains_of_alike_length_start_by_their_work(order):
    """Steps of 512 rows; a chain's calls follow each other in the order of the calls."""
    a, b = slices(2, 300, 0), slices(2, 320, 1)
    assert order("chains", [a[0], b[0], a[1], b[1]]) == [1, 3, 0, 2]
    assert order("chains", [(700, 700, 1, 0), (600, 9000, 1, 1)]) == [1, 0]
    assert order("chains", [(700, 700, 1, 0), (1024, 1024, 1, 1)]) == [1, 0]
