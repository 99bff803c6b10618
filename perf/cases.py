"""The work whose speed is tracked: chunked attention as a training program calls it, and the host planner.

Kinds of a case
  step   ChunkAttention over a planned batch: gradients cleared, forward over every chunk, backward over every chunk
         (K > 0: Algorithm 2 with K kept chunks, so that discarded chunks run forward again).  The plan, the tensors
         and the runner are what a training program holds when a layer's attention starts.
  fwd    one cf_attn_fwd call on one chunk, as a layer makes it between its projections.
  bwd    one cf_attn_bwd call on one chunk whose forward has run; dK / dV are added to, as behind later slices.
  plan   the host side of a new batch: chunk construction, Algorithm 2's schedule and the kernels' tile tables.

Lengths are drawn from the case alone (lens_seed), values N(0, 1) from the seed that prepare() is given.
"""
import math

import numpy as np
import torch

from paper_2503_02356_amd import binding as B
from paper_2503_02356_amd import inputs
from paper_2503_02356_amd.runner import ChunkAttention

DEV = "cuda:0"


def _step(name, dtype, Hq, Hkv, D, C, long_len, n_packed, median, K=0, merge=False, fused=False, lens_seed=0):
    """long_len > 0: one sequence of that many tokens, split into slices of C; n_packed: packed chunks' worth of short
    sequences, lognormal (sigma 0.9) around `median`."""
    c = dict(kind="step", dtype=dtype, Hq=Hq, Hkv=Hkv, D=D, C=C, long_len=long_len, n_packed=n_packed, median=median,
             K=K, merge=merge, fused=fused, lens_seed=lens_seed)
    return dict(c, name=name) if name else c


def _chunk(name, kind, dtype, Hq, Hkv, D, T, prefix, median, lens_seed=0):
    """One chunk of T query rows: median > 0: packed short sequences; median = 0: one slice behind `prefix` keys."""
    c = dict(kind=kind, dtype=dtype, Hq=Hq, Hkv=Hkv, D=D, T=T, prefix=prefix, median=median, lens_seed=lens_seed)
    return dict(c, name=name) if name else c


def _plan(name, n_seqs, C, long_share, K, merge, lens_seed=0):
    c = dict(kind="plan", n_seqs=n_seqs, C=C, long_share=long_share, K=K, merge=merge, lens_seed=lens_seed)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the fp32 configuration for checking a model in full precision: one head, 13 short calls; latency
        _step("tiny_fp32", "fp32", 1, 1, 64, 256, 700, 3, 60),
        # fp32, grouped heads, a split sequence among short ones: the same check at a model's head count
        _step("fp32_mixed", "fp32", 6, 2, 128, 1000, 2700, 3, 200),
        # bf16 models with 64-wide heads
        _step("d64_packed", "bf16", 16, 4, 64, 4096, 5000, 3, 300),
        # small micro-batches (the packed 8K configuration divided by 16): launches and host work count
        _step("packed_512", "bf16", 28, 4, 128, 512, 0, 16, 37),
        # one packed chunk, forward only (evaluation, activation recomputation)
        _chunk("packed_8k_fwd", "fwd", "bf16", 28, 4, 128, 8160, 0, 600),
        # the benchmark's batch: 16 packed chunks of 8192 tokens
        _step("packed_8k", "bf16", 28, 4, 128, 8192, 0, 16, 600),
        # the benchmark's second batch: a 32768-token sequence in 4 slices and 8 packed chunks
        _step("long32k_mixed", "bf16", 28, 4, 128, 8192, 32768, 8, 600),
        # Algorithm 2 at its smallest memory: one kept chunk, every other slice's forward runs twice
        _step("long32k_k1", "bf16", 28, 4, 128, 2048, 32768, 1, 600, K=1),
        # the long-tail configuration (32 / 8 heads, 16384), ragged, the last slice packed with short sequences
        _step("longtail_16k", "bf16", 32, 8, 128, 16384, 50001, 4, 800, merge=True),
        # a late slice of a very long sequence, forward and backward (64 / 8 heads, 32768-token slices)
        _chunk("long128k_fwd", "fwd", "bf16", 64, 8, 128, 32768, 98304, 0),
        _chunk("long128k_bwd", "bwd", "bf16", 64, 8, 128, 32768, 98304, 0),
        # planning the 20000-sequence batch
        _plan("plan_20000", 20000, 16384, 0.0011, 2, False),
    ]


_HEADS = [(28, 4), (32, 8), (64, 8), (16, 2), (8, 2), (4, 4), (14, 2), (32, 32)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; at most the arithmetic of long128k_bwd (bf16, 128-wide heads), or what the
    full-precision and 64-wide cases stand for (their sizes are those of checks and small models)."""
    seed = rng.randrange(1, 1 << 30)
    kind = rng.choice(["step", "step", "step", "small", "fwd", "bwd", "bwd", "plan"])
    while True:
        if kind == "step":
            Hq, Hkv = rng.choice(_HEADS)
            C = _log(rng, 256, 16384)
            slices = rng.choice([0, 0, rng.uniform(1.1, 5.0)])
            n_packed = rng.randint(1, 10)
            K = rng.choice([0, 0, 0, 1, 2])
            c = _step(None, "bf16", Hq, Hkv, 128, C, int(slices * C), n_packed, min(_log(rng, 40, 1500), C // 2), K=K,
                      merge=rng.random() < 0.25, fused=K == 0 and rng.random() < 0.25, lens_seed=seed)
            limit = 1.5e14
        elif kind == "small":
            dtype, D = rng.choice([("fp32", 64), ("fp32", 128), ("bf16", 64), ("bf16", 64)])
            Hq, Hkv = rng.choice([(1, 1), (4, 4), (6, 2), (8, 2), (16, 4)])
            C = _log(rng, 256, 4096)
            c = _step(None, dtype, Hq, Hkv, D, C, int(rng.choice([0, rng.uniform(1.1, 3.0)]) * C), rng.randint(1, 4),
                      min(_log(rng, 40, 600), C // 2), lens_seed=seed)
            limit = 2.0e11
        elif kind in ("fwd", "bwd"):
            Hq, Hkv = rng.choice(_HEADS)
            T = _log(rng, 100, 32768)
            packed = rng.random() < 0.4
            c = _chunk(None, kind, "bf16", Hq, Hkv, 128, T, 0 if packed else rng.choice([0, _log(rng, 100, 131072)]),
                       min(_log(rng, 40, 1500), max(1, T // 2)) if packed else 0, lens_seed=seed)
            limit = 2.5e14
        else:
            c = _plan(None, _log(rng, 100, 20000), _log(rng, 1024, 32768), rng.uniform(0.0, 0.01), rng.randint(1, 4),
                      rng.random() < 0.3, lens_seed=seed)
            return c
        if work(c)["flops"] <= limit:
            return c


# ---------------------------------------------------------------------------------------------------------------- sizes
def _short_lens(rng, median, hi, budget):
    """Lognormal lengths (sigma 0.9) in [1, hi] until the next one would exceed `budget` tokens."""
    lens, total = [], 0
    while True:
        n = int(min(max(1, round(float(rng.lognormal(math.log(median), 0.9)))), hi))
        if total + n > budget:
            return lens or [min(n, hi)]
        lens.append(n)
        total += n


def _batch_lens(case):
    """Sequence lengths of a step case: the split sequence first, then the short ones (1.5 % of the packed chunks'
    room is left free, so that the packing finds its bins)."""
    rng = np.random.default_rng([case["lens_seed"], 1])
    head = [case["long_len"]] if case["long_len"] > 0 else []
    return head + _short_lens(rng, case["median"], case["C"], int(case["n_packed"] * case["C"] * 0.985))


def _chunk_cu(case):
    """(cu_seqlens_q, cu_seqlens_k) of a single chunk."""
    T = case["T"]
    if case["median"] == 0:
        return np.array([0, T], np.int32), np.array([0, case["prefix"] + T], np.int32)
    lens = _short_lens(np.random.default_rng([case["lens_seed"], 2]), case["median"], T, T)
    if sum(lens) < T:
        lens.append(T - sum(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return cu, cu


def _plan_lens(case):
    rng = np.random.default_rng([case["lens_seed"], 3])
    n, C = case["n_seqs"], case["C"]
    n_long = max(1, round(case["long_share"] * n))
    short = np.clip(np.rint(rng.lognormal(math.log(800) - 0.405, 0.9, size=n - n_long)), 16, C)
    lens = np.concatenate([short, rng.integers(C + 1, 8 * C + 1, size=n_long)])
    rng.shuffle(lens)
    return lens.astype(np.int64)


def _build(lens, C, merge):
    return B.cf_build_chunks_ex(lens, C, B.CF_PLAN_MERGE_TAILS) if merge else B.cf_build_chunks(lens, C)


# ------------------------------------------------------------------------------------------------------------------ work
def work(case):
    """Arithmetic: 4 D per unmasked (query, key) pair and query head forward, 10 D backward (the five products of the
    gradient), what Algorithm 2 recomputes included.  Bytes: every tensor of a call once (gradients of keys and values
    read and written: they are added to)."""
    if case["kind"] == "plan":
        lens = _plan_lens(case)
        # a length in; sequence, start, length and cu_seqlens entry out per segment; a 32-byte record per query tile
        return {"bytes": float(8 * len(lens) + 24 * len(lens) + 32 * (int(lens.sum()) // 128)), "flops": float(20 * len(lens))}
    e = 2 if case["dtype"] == "bf16" else 4
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]

    def fwd(T, Tk, pairs):
        return 2 * T * Hq * D * e + 2 * Tk * Hkv * D * e + 4 * T * Hq, 4.0 * D * Hq * pairs

    def bwd(T, Tk, pairs):
        return 4 * T * Hq * D * e + 2 * Tk * Hkv * D * e + 4 * T * Hq + 2 * 2 * Tk * Hkv * D * 4, 10.0 * D * Hq * pairs
    if case["kind"] in ("fwd", "bwd"):
        cu_q, cu_k = _chunk_cu(case)
        lq, lk = np.diff(cu_q).astype(np.float64), np.diff(cu_k).astype(np.float64)
        by, fl = (fwd if case["kind"] == "fwd" else bwd)(int(cu_q[-1]), int(cu_k[-1]), float((lq * (lk - lq) + lq * (lq + 1) / 2).sum()))
        return {"bytes": float(by), "flops": float(fl)}
    C, K = case["C"], case["K"]
    by = fl = 0.0
    for n in _batch_lens(case):
        starts = list(range(0, n, C))
        for i, s in enumerate(starts):
            T = min(C, n - s)
            pairs = T * s + T * (T + 1) / 2
            runs = 2 if K and i < len(starts) - K else 1
            (b0, f0), (b1, f1) = fwd(T, s + T, pairs), bwd(T, s + T, pairs)
            by += runs * b0 + b1
            fl += runs * f0 + f1
        by += 2 * n * Hkv * D * 4                    # gradients cleared
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(case):
    """bf16: the parity bound on the relative 2-norm error (operands, P and dS in bf16, sums in fp32);
    fp32: 32-bit sums; the planner: whole numbers."""
    if case["kind"] == "plan":
        return "exact"
    return {"rel": 5e-3} if case["dtype"] == "bf16" else {"rel": 1e-5}


# --------------------------------------------------------------------------------------------------------------- program
def prepare(case, seed):
    if case["kind"] == "plan":
        # another seed: the same lengths in another order
        return {"case": case, "lens": np.random.default_rng([seed, 4]).permutation(_plan_lens(case))}
    Hq, Hkv, D, dtype = case["Hq"], case["Hkv"], case["D"], case["dtype"]
    if case["kind"] == "step":
        lens = _batch_lens(case)
        plan = _build(lens, case["C"], case["merge"])
        vals = lambda sid, L: inputs.seq_values_device(seed, sid, lens[sid], Hq, Hkv, D, dtype, DEV)
        eng = ChunkAttention(plan, Hq, Hkv, D, dtype, fused_launch=case["fused"]).load(vals)
        return {"case": case, "eng": eng}
    cu_q, cu_k = _chunk_cu(case)
    T, Tk = int(cu_q[-1]), int(cu_k[-1])
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    rand = lambda n, h: torch.randn((n, h, D), generator=gen, device=DEV, dtype=torch.float32).to(tdt)
    s = {"case": case, "o": torch.empty((T, Hq, D), dtype=tdt, device=DEV),
         "lse": torch.empty((Hq, T), dtype=torch.float32, device=DEV)}
    s["fwd"] = B.make_fwd_params(rand(T, Hq), rand(Tk, Hkv), rand(Tk, Hkv), s["o"], s["lse"], torch.from_numpy(cu_q).to(DEV),
                                 torch.from_numpy(cu_k).to(DEV), 1.0 / math.sqrt(D))
    if case["kind"] == "bwd":
        B.cf_attn_fwd(s["fwd"])
        s["dq"] = torch.empty((T, Hq, D), dtype=tdt, device=DEV)
        s["dk"] = torch.zeros((Tk, Hkv, D), dtype=torch.float32, device=DEV)
        s["dv"] = torch.zeros_like(s["dk"])
        ws = torch.empty(B.cf_attn_bwd_workspace_bytes(s["fwd"]), dtype=torch.uint8, device=DEV)
        s["bwd"] = B.make_bwd_params(s["fwd"], rand(T, Hq), s["dq"], s["dk"], s["dv"], ws)
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "fwd":
        B.cf_attn_fwd(state["fwd"])
        return {"o": state["o"], "lse": state["lse"]}
    if case["kind"] == "bwd":
        B.cf_attn_bwd(state["bwd"])
        return {"dq": state["dq"], "dk": state["dk"], "dv": state["dv"]}
    if case["kind"] == "step":
        eng = state["eng"]
        eng.zero_grads()
        if case["K"]:
            eng.run_schedule(case["K"])
        else:
            eng.run_forward()
            eng.run_backward()
        # dK / dV of every sequence live in one buffer, in plan order
        return {"o": [c["o"] for c in eng.chunks], "lse": [c["lse"] for c in eng.chunks],
                "dq": [c["d_q"] for c in eng.chunks], "dkv": eng.grad_arena}
    plan = _build(state["lens"], case["C"], case["merge"])
    ops = np.array(plan.schedule(case["K"]), dtype=np.int64)
    tiles = []
    for c in range(plan.n_chunks):
        cu_q = plan.chunk_cu_seqlens(c)
        if len(cu_q) == 2:
            cu_k = np.array([0, int(plan.chunk_prefix_len[c]) + int(cu_q[1])], dtype=np.int32)
        else:                                        # (a merged tail's keys are its whole sequence's)
            cu_k = np.concatenate([[0], np.cumsum([start + n for (_, start, n) in plan.chunk_segments(c)])]).astype(np.int32)
        tiles.append(B.cf_attn_q_tiles(cu_q, cu_k))
    return {"tokens": plan.chunk_tokens, "prefix": plan.chunk_prefix_len, "group": plan.chunk_group,
            "seq": plan.seg_seq_id, "start": plan.seg_seq_start, "len": plan.seg_len, "cu": plan.cu_seqlens,
            "chunks": plan.group_chunks, "ops": ops, "tiles": np.concatenate(tiles)}
