"""GPU parity at the sizes where a kernel or a dispatch rule changes its path: edges of tiles, remainders, the smallest
calls.  Reference: the fp64 oracle's unsplit attention; tolerances: tests/parity.py (per data type)."""
import numpy as np
import pytest
import torch

from paper_2503_02356_amd import binding as B
from paper_2503_02356_amd import inputs
from paper_2503_02356_amd.runner import ChunkAttention
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("lens,C,Hq,Hkv,scale", [
    ([1], 8, 1, 1, None),                                  # one row, one key
    ([15, 16, 17, 1, 2], 64, 3, 1, None),                  # around the 16-row block
    ([255, 256, 257, 270], 300, 2, 2, None),               # 16 blocks: one per wavefront; then a second round
    ([530], 100, 4, 2, None),                              # slices whose prefix is no multiple of 16
    ([70, 40], 32, 2, 1, -0.125), ([70, 40], 32, 2, 1, 0.0),   # any scale
])
def test_fp32_blocks(D, lens, C, Hq, Hkv, scale):
    got, _ = P.run_gpu(lens, C, Hq, Hkv, D, "fp32", seed=31, scale=scale)
    ref = P.run_oracle(lens, Hq, Hkv, D, "fp32", seed=31, scale=scale)
    P.check(got, ref, "fp32", f"lens={lens} C={C} D={D} scale={scale}")


@pytest.mark.parametrize("flags", [0, B.CF_FLAG_DKV_SINGLE_WRITER])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("lens,C,Hq,Hkv", [
    ([1], 8, 1, 1),                                        # one row, one key: one wavefront of four has keys
    ([31, 32, 33, 63, 64, 65, 127, 128, 129], 642, 4, 2),  # around a wavefront's keys, a query tile, a key tile
    ([1 + i % 3 for i in range(300)], 600, 2, 1),          # more segments than the work list is built from at once
    ([700], 70, 7, 1),                                     # slices that start inside a sequence's first 128 positions
    ([2500], 1300, 8, 1),                                  # key tiles whose query heads are split over work items
])
def test_bf16_blocks(D, lens, C, Hq, Hkv, flags):
    got, _ = P.run_gpu(lens, C, Hq, Hkv, D, "bf16", seed=32, flags=flags)
    ref = P.run_oracle(lens, Hq, Hkv, D, "bf16", seed=32)
    P.check(got, ref, "bf16", f"lens={lens[:9]} C={C} D={D} flags={flags}")


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (3, 1), (5, 1), (14, 2)])
@pytest.mark.parametrize("lens,C", [([1, 31, 32, 33, 64, 65, 96, 97, 129, 161], 709), ([333], 100)])
def test_blocks_of_a_group_dealt_to_four_wavefronts(lens, C, Hq, Hkv):
    """dK/dV at D = 64: the 32-row blocks of all heads of a group go round four wavefronts: fewer blocks than wavefronts, heads of fewer
    blocks than a round, a last block of one row, slices whose blocks start behind the keys."""
    got, _ = P.run_gpu(lens, C, Hq, Hkv, 64, "bf16", seed=37)
    P.check(got, P.run_oracle(lens, Hq, Hkv, 64, "bf16", seed=37), "bf16", f"lens={lens} C={C} heads={Hq}/{Hkv}")


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("lens,C,Hq,Hkv", [([300, 41, 700, 64, 9, 150], 256, 4, 2), ([40] * 30 + [130] * 5, 600, 2, 2)])
def test_errors_are_no_larger_than_the_scalar_kernels(dtype, D, lens, C, Hq, Hkv):
    """Shapes whose P, dS and sums are fp32 in the scalar kernels: relative 2-norm error against the fp64 oracle, per tensor.
    5 %: how far the errors of two sums of equal precision over these few thousand elements may lie apart."""
    ref = P.run_oracle(lens, Hq, Hkv, D, dtype, seed=34)
    here, scalar = (P.errors(P.run_gpu(lens, C, Hq, Hkv, D, dtype, seed=34, flags=f)[0], ref) for f in (0, B.CF_FLAG_SCALAR_KERNELS))
    for n in P.NAMES:
        assert here[n][1] <= 1.05 * scalar[n][1], (n, here[n], scalar[n])


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("fp32", 64), ("fp32", 128)])
def test_calls_that_share_launches(dtype, D):
    """A list of calls (more than one launch holds; slices of one sequence, whose gradients meet, among them) against the
    same calls one at a time: O, LSE, dQ bit for bit; dK/dV too in fp32, in bf16 (atomic adds) to fp32 rounding."""
    lens = [500, 40, 130, 77, 9, 128, 33, 100, 64, 90, 41, 127, 5, 120, 88, 110, 101, 99, 97, 95]
    got, eng = P.run_gpu(lens, 130, 4, 2, D, dtype, seed=33)
    assert len(eng.chunks) > 16
    P.check(got, P.run_oracle(lens, 4, 2, D, dtype, seed=33), dtype, "calls")
    eng.zero_grads()
    for c in eng.forward_order():
        B.cf_attn_fwd(eng.chunks[c]["fwd"])
    for c in eng.backward_order():
        B.cf_attn_bwd(eng.chunks[c]["bwd"])
    one = eng.results()
    for sid in got:
        for n in P.NAMES:
            a, b = got[sid][n], one[sid][n]
            if n in ("dk", "dv") and dtype == "bf16":      # at most 40 additions, each rounded to 2^-24 of a partial sum (up to 4x the result)
                assert np.abs(a - b).max() <= 40 * 2.0 ** -24 * max(1.0, np.abs(b).max()) * 4, (sid, n)
            else:
                assert np.array_equal(a, b), (sid, n)


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("lens,C,Hq,Hkv", [
    ([1100, 31, 33, 64, 65, 127, 129, 4, 300], 500, 8, 2),     # keys and rows around a workgroup's, slices of one sequence, head groups
    ([2300], 2300, 8, 1),                                      # many query tiles per key tile: work that invites a split over heads
])
def test_gradients_repeat_bitwise(dtype, D, lens, C, Hq, Hkv):
    """One writer per dK/dV row without any flag: a second pass, and the same calls one at a time, give the same bits."""
    got, eng = P.run_gpu(lens, C, Hq, Hkv, D, dtype, seed=35)

    def again(backward):
        eng.zero_grads()
        backward()
        return eng.results()
    for backward in (eng.run_backward, lambda: [B.cf_attn_bwd(eng.chunks[c]["bwd"]) for c in eng.backward_order()]):
        r = again(backward)
        for sid in got:
            for n in ("dq", "dk", "dv"):
                assert np.array_equal(got[sid][n], r[sid][n]), (sid, n)


@pytest.mark.parametrize("dtype,D,flags,merge", [("bf16", 128, 0, False), ("bf16", 128, 0, True), ("bf16", 128, B.CF_FLAG_DKV_SINGLE_WRITER, False),
                                                 ("bf16", 64, 0, False), ("fp32", 64, 0, False), ("fp32", 128, 0, True)])
def test_slices_that_add_to_the_same_rows(dtype, D, flags, merge):
    """The slices of split sequences add to the same rows of dK and dV, in a list of calls as one by one.  What is added is the same
    up to the order of fp32 sums: fewer than 64 terms to an element, 64 * 2^-24 = 4e-6."""
    lens, C, Hq, Hkv = [700, 30, 530, 61, 129, 90], 256, 4, 2
    plan = B.cf_build_chunks_ex(lens, C, B.CF_PLAN_MERGE_TAILS) if merge else B.cf_build_chunks(lens, C)
    vals = lambda sid, L: inputs.seq_values(5, sid, L, Hq, Hkv, D, dtype)
    eng = ChunkAttention(plan, Hq, Hkv, D, dtype, flags=flags).load(vals)
    results = []
    for together in (False, True):
        eng.grad_arena.normal_(generator=torch.Generator(device="cuda:0").manual_seed(1))       # (they are added to)
        eng.run_forward()
        if together:
            eng.run_backward()
        else:
            for c in eng.backward_order():
                B.cf_attn_bwd(eng.chunks[c]["bwd"])
        torch.cuda.synchronize()
        results.append((eng.grad_arena.clone(), [ch["d_q"].clone() for ch in eng.chunks]))
    (g0, q0), (g1, q1) = results
    assert all(torch.equal(a, b) for a, b in zip(q0, q1))
    assert ((g0 - g1).norm() / g0.norm()).item() <= 64 * 2.0 ** -24


@pytest.mark.parametrize("Hq,Hkv,C,merge", [(4, 4, 128, False), (4, 2, 64, False), (4, 4, 128, True), (8, 8, 100, False)])
@pytest.mark.parametrize("backwards", [False, True])
def test_one_work_item_to_a_key_tile_adds_in_the_order_of_the_calls(Hq, Hkv, C, merge, backwards):
    """bf16, D = 128: where every call adds once to a row of dK and dV, the sums over the slices of a sequence have the bits of
    separate calls, whatever shares their launches."""
    lens = [11 * C + 37, 30, 7 * C, 61, 5 * C + 1, 20]
    plan = B.cf_build_chunks_ex(lens, C, B.CF_PLAN_MERGE_TAILS) if merge else B.cf_build_chunks(lens, C)
    eng = ChunkAttention(plan, Hq, Hkv, 128, "bf16").load(lambda sid, L: inputs.seq_values(9, sid, L, Hq, Hkv, 128, "bf16"))
    eng.run_forward()
    order = eng.backward_order()[::-1] if backwards else eng.backward_order()
    ws = [torch.empty_like(eng.workspaces[0]) for _ in order]
    calls = [B.make_bwd_params(c["fwd"], c["d_o"], c["d_q"], c["dk"], c["dv"], w) for c, w in zip((eng.chunks[c] for c in order), ws)]
    got = []
    for together in (False, True, True, True):
        eng.grad_arena.normal_(generator=torch.Generator(device="cuda:0").manual_seed(1))       # (they are added to)
        if together:
            B.cf_attn_calls(B.make_calls((True, b) for b in calls))
        else:
            for b in calls:
                B.cf_attn_bwd(b)
        torch.cuda.synchronize()
        got.append(eng.grad_arena.clone())
    assert all(torch.equal(got[0], g) for g in got[1:])


def _together_and_apart(calls, grads):
    """Gradient buffers and dQ of backward calls in one list and one at a time, on the same start values."""
    got = []
    for together in (False, True):
        for i, g in enumerate(grads):
            g.normal_(generator=torch.Generator(device="cuda:0").manual_seed(i))        # (they are added to)
        if together:
            B.cf_attn_calls(B.make_calls((True, b) for b in calls))
        else:
            for b in calls:
                B.cf_attn_bwd(b)
        torch.cuda.synchronize()
        got.append([g.clone() for g in grads] + [b._keepalive[2].clone() for b in calls])
    return got


def _calls_of(eng, order, grads=lambda ch: (ch["dk"], ch["dv"])):
    ch = [eng.chunks[c] for c in order]
    return [B.make_bwd_params(c["fwd"], c["d_o"], c["d_q"], *grads(c), torch.empty_like(eng.workspaces[0])) for c in ch]


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("backwards", [False, True])
@pytest.mark.parametrize("merge", [False, True])
def test_chains_of_slices_keep_the_bits_of_single_calls(dtype, D, backwards, merge):
    """Split sequences and packed chunks, 22 backward calls (two launches, a chain cut between them): slices that end inside a
    block of 16 or 32 keys, the first call of a chain its longest or its shortest one, last slices in packed chunks (which add to
    rows of a chain and are none of it).  Same bits as one call at a time."""
    lens, C, Hq, Hkv = [333, 210, 20, 71, 130, 9, 64, 290, 65, 33, 100], 70, 4, 2
    plan = B.cf_build_chunks_ex(lens, C, B.CF_PLAN_MERGE_TAILS) if merge else B.cf_build_chunks(lens, C)
    vals = lambda sid, L: inputs.seq_values(8, sid, L, Hq, Hkv, D, dtype)
    eng = ChunkAttention(plan, Hq, Hkv, D, dtype).load(vals)
    eng.run_forward()
    order = eng.backward_order()[::-1] if backwards else eng.backward_order()
    assert len(order) > B.BWD_TOGETHER and sum(len(plan.group(g)) > 2 for g in eng.groups()) >= 3
    first = (len(order) + 1) // 2                    # (two launches of equal size, where nothing else ends the first one)
    assert merge or any(set(plan.group(g)) & set(order[:first]) and set(plan.group(g)) & set(order[first:]) for g in eng.groups())
    assert merge == any(ch["merged"] for ch in eng.chunks)
    apart, together = _together_and_apart(_calls_of(eng, order), [eng.grad_arena])
    assert all(torch.equal(a, b) for a, b in zip(apart, together))


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("name,value", [("q", float("nan")), ("d_o", float("inf")), ("v", float("-inf")), ("k", float("nan"))])
def test_chains_take_rows_again_that_are_not_finite(dtype, D, name, value):
    """A value that is not finite in the third of five slices, dK and dV as views into one buffer: the rows that the matrix product
    leaves out of a slice's gradients are added pair by pair between two slices of the chain.  Same bits as one call at a time."""
    L, C, Hq, Hkv = 333, 70, 4, 2
    plan = B.cf_build_chunks([L], C)
    eng = ChunkAttention(plan, Hq, Hkv, D, dtype).load(lambda sid, n: inputs.seq_values(8, sid, n, Hq, Hkv, D, dtype))
    where = eng.chunks[2]
    (where[name][where["P"] + 33] if name in "kv" else where[name][33])[1, 5] = value
    eng.run_forward()
    both = torch.empty(L, Hkv, 2, D, device="cuda:0")
    calls = _calls_of(eng, eng.backward_order(), lambda ch: tuple(both[:len(ch["k"]), :, i] for i in (0, 1)))
    apart, together = _together_and_apart(calls, [both])
    bad = ~torch.isfinite(apart[0])
    assert bad.any() and not bad.all()
    for a, b in zip(apart, together):
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(nan=0.), b.nan_to_num(nan=0.))


@pytest.mark.parametrize("Hq,Hkv,C", [(4, 4, 128), (8, 2, 256)])
def test_single_writers_among_work_lists(Hq, Hkv, C):
    """bf16, D = 128, slices of one sequence: calls with one writer per dK/dV row next to calls with work lists.  One head per
    group: every call adds once to a row, same bits as one call at a time; else up to the order of fp32 sums (as above)."""
    plan = B.cf_build_chunks([6 * C + 50, 40, 5 * C, 61], C)
    eng = ChunkAttention(plan, Hq, Hkv, 128, "bf16").load(lambda sid, L: inputs.seq_values(7, sid, L, Hq, Hkv, 128, "bf16"))
    eng.run_forward()
    calls = _calls_of(eng, eng.backward_order())
    for i, b in enumerate(calls):
        b.f.flags = B.CF_FLAG_DKV_SINGLE_WRITER if i % 3 == 1 else 0
    apart, together = _together_and_apart(calls, [eng.grad_arena])
    assert all(torch.equal(a, b) for a, b in zip(apart[1:], together[1:]))
    if Hq == Hkv:
        assert torch.equal(apart[0], together[0])
    else:
        assert ((apart[0] - together[0]).norm() / apart[0].norm()).item() <= 64 * 2.0 ** -24


@pytest.mark.parametrize("Hq,Hkv,C", [(8, 2, 512), (8, 2, 513), (4, 4, 1024), (28, 4, 146), (28, 4, 147)])
def test_both_sizes_of_mfma(Hq, Hkv, C):
    """bf16, D = 128: calls of up to 4096 (query row, head) pairs use 32x32x16 MFMAs in the forward and dQ, others 16x16x32.  Lists of calls
    with the one, the other and both give the bits of single calls, and match the oracle."""
    lens = [2 * C + 45, 30, C - 1, 61, 20]
    plan = B.cf_build_chunks(lens, C)
    vals = lambda sid, L: inputs.seq_values(6, sid, L, Hq, Hkv, 128, "bf16")
    eng = ChunkAttention(plan, Hq, Hkv, 128, "bf16").load(vals)
    small = [ch["T"] * Hq <= 4096 for ch in eng.chunks]
    assert any(small) and all(small) == (C * Hq <= 4096)
    res = []
    for one_by_one in (True, False):
        eng.zero_grads()
        if one_by_one:
            for c in eng.forward_order():
                B.cf_attn_fwd(eng.chunks[c]["fwd"])
            for c in eng.backward_order():
                B.cf_attn_bwd(eng.chunks[c]["bwd"])
        else:
            eng.run_forward(), eng.run_backward()
        res.append(eng.results())
        P.check(res[-1], P.run_oracle(lens, Hq, Hkv, 128, "bf16", seed=6), "bf16", f"one by one: {one_by_one}")
    for sid in res[0]:
        for n in ("o", "lse", "dq"):
            assert np.array_equal(res[0][sid][n], res[1][sid][n]), (sid, n)


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("fp32", 64)])
def test_results_do_not_depend_on_the_order_in_a_launch(dtype, D):
    """A list whose launches start with its last call (tests/test_launch_order.py): the last slice of the split sequence, 20 rows behind 600
    keys, has the longest chain and the least work.  Same bits of O, LSE and dQ as one call at a time, and the oracle's results."""
    lens, C, Hq, Hkv = [620, 150, 140, 10, 130, 100, 70], 300, 4, 2
    got, eng = P.run_gpu(lens, C, Hq, Hkv, D, dtype, seed=35)
    work = {c: ch["T"] * (ch["P"] + ch["T"]) for c, ch in enumerate(eng.chunks)}
    tail = [c for c, ch in enumerate(eng.chunks) if ch["P"] == 600]
    assert len(tail) == 1 and work[tail[0]] == min(work.values())
    P.check(got, P.run_oracle(lens, Hq, Hkv, D, dtype, seed=35), dtype, "list")
    eng.zero_grads()
    for c in eng.forward_order():
        B.cf_attn_fwd(eng.chunks[c]["fwd"])
    for c in eng.backward_order():
        B.cf_attn_bwd(eng.chunks[c]["bwd"])
    one = eng.results()
    for sid in got:
        for n in ("o", "lse", "dq"):
            assert np.array_equal(got[sid][n], one[sid][n]), (sid, n)


@pytest.mark.parametrize("dtype,D,one_slot", [("bf16", 128, False), ("bf16", 128, True), ("bf16", 64, True), ("fp32", 64, False), ("fp32", 64, True)])
def test_forward_and_backward_in_turns(dtype, D, one_slot):
    """Algorithm 2 with one kept chunk, as a list: calls move past others that they have nothing to do with.  Same results as one call at
    a time (dK/dV: up to the order of at most 40 fp32 sums where items meet in atomic adds), also where all chunks share one O and one LSE,
    so that each backward has to come between its forward and the next one.  Two heads' sizes: the kernels alternate too."""
    C, results = 130, []
    engines = []
    for Hq, lens in ((4, [700, 60, 129, 40, 30]), (2, [390, 131])):
        plan = B.cf_build_chunks(lens, C)
        eng = ChunkAttention(plan, Hq, 2, D, dtype).load(lambda sid, L: inputs.seq_values(11, sid, L, Hq, 2, D, dtype))
        engines.append((plan, eng, [(op == B.CF_OP_BWD, c) for op, c in plan.schedule(1)]))
    if one_slot:
        for plan, eng, _ in engines:
            for c in range(plan.n_chunks):
                ch = eng.chunks[c]
                o, lse = eng.chunks[0]["o"], eng.chunks[0]["lse"]
                assert ch["T"] <= o.shape[0]
                ch["o"], ch["lse"] = o[:ch["T"]], lse.view(-1)[:lse.shape[0] * ch["T"]].view(lse.shape[0], ch["T"])
                ch["fwd"] = B.make_fwd_params(ch["q"], ch["k"], ch["v"], ch["o"], ch["lse"], ch["cu_q"], ch["cu_k"], eng.scale)
                ch["bwd"] = B.make_bwd_params(ch["fwd"], ch["d_o"], ch["d_q"], ch["dk"], ch["dv"], torch.empty_like(eng.workspaces[0]))
    (_, e0, ops0), (_, e1, ops1) = engines
    ops = [(e, *op) for pair in zip(ops0, ops1) for e, op in zip((e0, e1), pair)] + [(e0, *op) for op in ops0[len(ops1):]]
    assert len(ops1) <= len(ops0) and len(ops) < 64 and sum(bwd for _, bwd, _ in ops) > 8
    calls = [(bwd, e.chunks[c]["bwd" if bwd else "fwd"]) for e, bwd, c in ops]
    for together in (False, True, True):
        for e in (e0, e1):
            e.grad_arena.zero_()
            for ch in e.chunks:
                ch["o"].fill_(float("nan")), ch["lse"].fill_(float("nan")), ch["d_q"].fill_(float("nan"))
        if together:
            B.cf_attn_calls(B.make_calls(calls))
        else:
            for bwd, params in calls:
                (B.cf_attn_bwd if bwd else B.cf_attn_fwd)(params)
        torch.cuda.synchronize()
        results.append([t.clone() for e in (e0, e1) for ch in e.chunks for t in (ch["d_q"], ch["o"], ch["lse"])] + [e.grad_arena.clone() for e in (e0, e1)])
    for got in results[1:]:
        assert all(torch.equal(a, b) for a, b in zip(results[0][:-2], got[:-2]))
        for a, b in zip(results[0][-2:], got[-2:]):
            assert torch.equal(a, b) if (dtype, D) != ("bf16", 128) else ((a - b).norm() / a.norm()).item() <= 40 * 2.0 ** -24


@pytest.mark.parametrize("Hq,T", [(32, 130), (4, 130), (32, 300)])
@pytest.mark.parametrize("together", [False, True])
def test_dp_is_summed_before_delta_is_taken_off(Hq, T, together):
    """dQ at D = 128, both sizes of MFMA: of delta = -1 and dP = 2^-8 + 4 x 2^-25, a 2^-25 from every 32 columns, dP - delta is
    1 + 2^-8 + 2^-23, which fp32 holds and which rounds up to the bf16 1 + 2^-7.  A sum that starts at -delta loses each 2^-25 and is left
    with 1 + 2^-8, half way, which rounds to 1.  Q = 0 and LSE = 0 make every P 1, one key's K = 1 brings its dS into dQ; the rows are far
    enough from the start of the sequence for delta to be <dO, O>."""
    D, prefix, bf16 = 128, 200, torch.bfloat16
    dev = lambda *shape, dtype=bf16, value=0: torch.full(shape, value, dtype=dtype, device="cuda:0")
    q, o, d_o, k, v = dev(T, Hq, D), dev(T, Hq, D), dev(T, Hq, D, value=1), dev(prefix + T, 4, D), dev(prefix + T, 4, D)
    o[:, :, 0] = -1
    k[5, :, 0] = 1
    v[5, :, 0] = 2.0 ** -8
    v[5, :, 1::32] = 2.0 ** -25
    lse, dq, dkv = dev(Hq, T, dtype=torch.float32), dev(T, Hq, D), dev(2, prefix + T, 4, D, dtype=torch.float32)
    cu = [torch.tensor([0, n], dtype=torch.int32, device="cuda:0") for n in (T, prefix + T)]
    f = B.make_fwd_params(q, k, v, o, lse, *cu, 1.0)
    calls = []
    for _ in range(2 if together else 1):
        ws = torch.empty(B.cf_attn_bwd_workspace_bytes(f), dtype=torch.uint8, device="cuda:0")
        calls.append((True, B.make_bwd_params(f, d_o, torch.full_like(dq, float("nan")), dkv[0], dkv[1], ws)))
    B.cf_attn_calls(B.make_calls(calls))
    torch.cuda.synchronize()
    want = dev(T, Hq, D)
    want[:, :, 0] = 1 + 2.0 ** -7
    for _, b in calls:
        assert torch.equal(b._keepalive[2], want)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_calls_that_depend_on_each_other(dtype):
    """The second forward takes the first one's output as its queries; the list stops at a call that is refused."""
    dt, T, H, D = torch.bfloat16 if dtype == "bf16" else torch.float32, 200, 2, 128
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    rand = lambda: torch.randn(T, H, D, device="cuda:0", generator=gen).to(dt)
    q, k, v, cu = rand(), rand(), rand(), torch.tensor([0, 77, T], dtype=torch.int32, device="cuda:0")
    o = [torch.zeros_like(q) for _ in range(3)]
    lse = [torch.zeros(H, T, device="cuda:0") for _ in range(3)]
    f = [B.make_fwd_params(a, k, v, o[i], lse[i], cu, cu, 0.09) for i, a in enumerate((q, o[0], q))]
    for p in f[:2]:
        B.cf_attn_fwd(p)
    want = o[1].clone()
    o[0].zero_(), o[1].zero_()
    f[2].n_segments = 0
    B.cf_attn_calls(B.make_calls([]))
    with pytest.raises(B.CfError):
        B.cf_attn_calls(B.make_calls((False, p) for p in f))
    torch.cuda.synchronize()
    assert torch.equal(o[1], want) and not o[2].any()


def _backward(q, k, v, d_o, flags=0, workspace_bytes=None):
    """-> o, lse, dq, dk, dv of one packed chunk of two segments."""
    (T, H, D), Hkv, dev = q.shape, k.shape[1], q.device
    o, dq, lse = torch.empty_like(d_o.contiguous()), torch.empty_like(d_o.contiguous()), torch.zeros(H, T, device=dev)
    dkv = torch.zeros(2, T, Hkv, D, device=dev)
    cu = torch.tensor([0, T // 3, T], dtype=torch.int32, device=dev)
    fp = B.make_fwd_params(q, k, v, o, lse, cu, cu, D ** -0.5, flags)
    B.cf_attn_fwd(fp)
    ws = torch.empty(workspace_bytes or B.cf_attn_bwd_workspace_bytes(fp), dtype=torch.uint8, device=dev)
    B.cf_attn_bwd(B.make_bwd_params(fp, d_o, dq, dkv[0], dkv[1], ws))
    torch.cuda.synchronize()
    return o, lse, dq, dkv[0], dkv[1]


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("lens,prefix,where", [
    ([150, 200], 0, 70), ([150, 200], 0, 149), ([150, 200], 0, 155),      # in a block's middle, a segment's last row, another's first ones
    ([90], 100, 130), ([300], 0, 299),
])
def test_infinities_and_nans_reach_only_the_rows_that_see_them(dtype, D, lens, prefix, where):
    """An infinity in V, a NaN in K, Q or dO, at row `where` of the keys (queries: of the same token): the scalar kernels never
    read a pair that the mask hides, so what is finite there has to be finite here, and agree."""
    dt, T, Hq, Hkv = torch.bfloat16 if dtype == "bf16" else torch.float32, sum(lens), 4, 2
    gen = torch.Generator(device="cuda:0").manual_seed(8)
    rand = lambda n, h: torch.randn(n, h, D, device="cuda:0", generator=gen).to(dt)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cu_k = cu + (np.arange(len(cu)) > 0) * np.int32(prefix)
    cu, cu_k = (torch.from_numpy(a).to("cuda:0") for a in (cu, cu_k))
    clean = rand(T, Hq), rand(T + prefix, Hkv), rand(T + prefix, Hkv), rand(T, Hq)
    for n, value in ((1, float("nan")), (2, float("inf")), (0, float("nan")), (3, float("nan")), (3, float("-inf"))):
        q, k, v, d_o = t = [x.clone() for x in clean]
        t[n][where - (prefix if n in (0, 3) else 0), 1, 5] = value
        res = []
        for flags in (0, B.CF_FLAG_SCALAR_KERNELS):
            o, dq, lse = torch.empty_like(q), torch.empty_like(q), torch.empty(Hq, T, device="cuda:0")
            dk, dv = torch.zeros(T + prefix, Hkv, D, device="cuda:0"), torch.zeros(T + prefix, Hkv, D, device="cuda:0")
            f = B.make_fwd_params(q, k, v, o, lse, cu, cu_k, D ** -0.5, flags)
            B.cf_attn_fwd(f)
            ws = torch.empty(B.cf_attn_bwd_workspace_bytes(f), dtype=torch.uint8, device="cuda:0")
            B.cf_attn_bwd(B.make_bwd_params(f, d_o, dq, dk, dv, ws))
            torch.cuda.synchronize()
            res.append((o, lse, dq, dk, dv))
        for name, a, b in zip(P.NAMES, *res):
            fine = torch.isfinite(b)
            assert torch.equal(torch.isfinite(a), fine), (n, value, name)
            d, r = (a[fine].double() - b[fine].double()).norm(), b[fine].double().norm()
            assert d <= P.TOL[dtype][1] * r, (n, value, name, float(d / r))


@pytest.mark.parametrize("lens,prefix,Hq,Hkv,least", [
    ([900, 300, 2100, 37, 128, 640, 1500, 555, 1000, 64, 968], 0, 28, 4, False),   # a packed chunk of 8192 tokens
    ([4000], 0, 4, 4, False),                              # one head per group: nothing to split but its query tiles
    ([130], 3000, 8, 2, False), ([16384], 0, 8, 1, False), # a short slice behind a prefix; a long sequence
    ([1500, 200, 40], 100, 14, 2, False), ([1] * 700, 0, 8, 2, False), ([3000] * 3, 0, 28, 4, False),
    ([4000], 0, 4, 4, True), ([1] * 300, 0, 2, 1, True),   # a scratch with room for G items per key tile only
])
def test_dkv_work_list(lens, prefix, Hq, Hkv, least):
    """The list a bf16 backward leaves in its scratch: every (head, query tile) pair of every key tile in exactly one item, longest
    items first, none longer than 1.6 times what one of 512 slots gets on average (small calls: 1.6 x 2.2) nor more items
    than that asks for."""
    T, Tk, G, D = sum(lens), sum(lens) + prefix, Hq // Hkv, 128
    t = lambda n, h: torch.randn(n, h, D, device="cuda:0").bfloat16()
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cu_k = cu + (np.arange(len(cu)) > 0) * np.int32(prefix)
    dev = lambda a: torch.from_numpy(a).to("cuda:0")
    q, k = t(T, Hq), t(Tk, Hkv)
    f = B.make_fwd_params(q, k, k, torch.empty_like(q), torch.empty(Hq, T, device="cuda:0"), dev(cu), dev(cu_k), D ** -0.5)
    delta = (Hq * T * 4 + 255) // 256 * 256
    n_bytes = B.cf_attn_bwd_workspace_bytes(f)
    if least:
        n_bytes = min(n_bytes, delta + 256 + 16 * G * (Tk // 128 + len(lens)))
    ws = torch.zeros(n_bytes, dtype=torch.uint8, device="cuda:0")
    dk, dv = torch.zeros(Tk, Hkv, D, device="cuda:0"), torch.zeros(Tk, Hkv, D, device="cuda:0")
    B.cf_attn_fwd(f)
    B.cf_attn_bwd(B.make_bwd_params(f, q, torch.empty_like(q), dk, dv, ws))
    wl = ws[delta:].cpu().numpy().view(np.int32)
    items = wl[64:64 + 4 * wl[0]].reshape(-1, 4).tolist()

    pairs = {}
    for g, lq in enumerate(lens):
        off = int(cu_k[g + 1] - cu_k[g]) - lq
        for kt in range(0, lq + off, 128):
            n = -(-lq // 64) - max(0, kt - off) // 64
            if n > 0:
                pairs[g, kt] = G * n
    seen = {}
    for g, kt, first, n in sorted(items):
        assert n > 0 and first == seen.get((g, kt), 0)
        seen[g, kt] = first + n
    assert seen == pairs
    length = [min(n, 255) for *_, n in items]
    assert length == sorted(length, reverse=True)
    average = sum(pairs.values()) * Hkv / 512
    most = max(3, np.ceil(average * 2.2)) * 1.6 if average <= 8 else np.ceil(average * 1.6)
    if least:
        assert len(items) <= G * len(pairs)
    else:
        assert length[0] <= most or average > 40          # (long sequences: whole heads of up to 255 and more)
        assert len(items) <= max(G * len(pairs), len(pairs) + 320 // Hkv + 1)


def test_d64_backward_without_room_for_a_work_list():
    """bf16, head_dim 64, a workspace that holds delta and nothing else (all that is asked for): the single-writer kernel, bit
    for bit."""
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    rand = lambda h: torch.randn(600, h, 64, device="cuda:0", generator=gen).bfloat16()
    t = rand(4), rand(2), rand(2), rand(4)
    least = (4 * 600 * 4 + 255) // 256 * 256
    for a, b in zip(_backward(*t, workspace_bytes=least), _backward(*t, flags=B.CF_FLAG_DKV_SINGLE_WRITER)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,T,Hq,n_calls", [("fp32", 70000, 64, 1), ("bf16", 270000, 64, 1), ("fp32", 30000, 64, 3), ("bf16", 100000, 64, 3)])
def test_more_segments_than_one_launch_holds(dtype, T, Hq, n_calls):
    """One-token sequences, D = 64: more workgroups than one launch holds (2^32 work-items), in one call or in calls that would
    share a launch.  O = V, LSE = the scaled score, dQ = dK = 0, dV = dO of the head group, all but exactly."""
    dt, D, dev = torch.bfloat16 if dtype == "bf16" else torch.float32, 64, "cuda:0"
    gen = torch.Generator(device=dev).manual_seed(9)
    rand = lambda h: torch.randn(T, h, D, device=dev, generator=gen).to(dt)
    cu = torch.arange(T + 1, dtype=torch.int32, device=dev)
    q, k, v, d_o = rand(Hq), rand(1), rand(1), rand(Hq)
    calls, bwd, out = [], [], []
    for _ in range(n_calls):
        o, dq, lse, dkv = torch.zeros_like(q), torch.ones_like(q), torch.zeros(Hq, T, device=dev), torch.zeros(2, T, 1, D, device=dev)
        f = B.make_fwd_params(q, k, v, o, lse, cu, cu, D ** -0.5)
        ws = torch.empty(B.cf_attn_bwd_workspace_bytes(f), dtype=torch.uint8, device=dev)
        calls.append((False, f))
        bwd.append((True, B.make_bwd_params(f, d_o, dq, dkv[0], dkv[1], ws)))
        out.append((o, lse, dq, dkv))
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    B.cf_attn_calls(B.make_calls(calls + bwd))
    end.record()
    torch.cuda.synchronize()
    assert start.elapsed_time(end) < 2500                  # ms; 100 to 400 measured (a search that grows with the segments: up to 15 s)
    score = torch.stack([(q[:, h].float() * k[:, 0].float()).sum(-1) * D ** -0.5 for h in range(Hq)])
    dv = sum(d_o[:, h].float() for h in range(Hq))
    for o, lse, dq, dkv in out:
        assert (o - v).abs().max() <= 2.0 ** -22 * v.abs().max()
        assert (lse - score).abs().max() <= 64 * 2.0 ** -24 * 8          # a sum of 64 products of a few units each
        assert dq.abs().max() <= 1e-4 and dkv[0].abs().max() <= 1e-3      # P - 1, rounded, times |dP| ~ 8 (64 heads)
        assert (dkv[1][:, 0] - dv).abs().max() <= 1e-4                    # 64 terms, rounded


@pytest.mark.parametrize("wide", ["q", "kv", "do"])
def test_strides_beyond_32_bit_offsets(wide):
    """64 rows of 2^25 bf16 elements span 4 GiB, more than the matrix kernels' row offsets: the results of the scalar
    kernels (of each pass that the wide tensor is an input of), bit for bit."""
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    T, D, stride = 70, 64, 1 << 25
    rand = lambda: torch.randn(T, 1, D, device="cuda:0", generator=gen).bfloat16()
    q, k, v, d_o = rand(), rand(), rand(), rand()
    room = torch.empty((T - 1) * stride + 2 * D, dtype=torch.bfloat16, device="cuda:0")

    def spread(x, at):
        y = room[at:].as_strided((T, 1, D), (stride, D, 1))
        return y.copy_(x)
    want = _backward(q, k, v, d_o, flags=B.CF_FLAG_SCALAR_KERNELS)
    got = _backward(spread(q, 0) if wide == "q" else q, spread(k, 0) if wide == "kv" else k, spread(v, D) if wide == "kv" else v,
                    spread(d_o, 0) if wide == "do" else d_o)
    for n, a, b in zip(("o", "lse", "dq", "dk", "dv"), got, want):
        if wide == "do":        # its forward ran on the matrix kernels: bf16 results within their rounding
            assert (a.double() - b.double()).norm() <= 5e-3 * b.double().norm(), n
        else:
            assert torch.equal(a, b), n
