"""The work this library does for its users, as cases that can be timed and compared.

A case is one call sequence over one packed batch.  Four kinds occur in a training program:

  step        routing scores -> top-k selection -> work plan -> attention forward -> attention backward, the whole path
              of one training step (the score matrix is kept: the budget controller reads it)
  forward     the same without the backward, scores and selection in one call that keeps no score matrix: a pass
              over evaluation data
  controller  routing scores -> coverage curves (what the budget controller decides on) -> selection
  sink        plan -> forward -> backward for a selection that the caller brings, with the shape real attention maps
              have: every query block keeps block 0 and the blocks right before it

The lengths of a batch come from `mix`:
  one         one sequence of `tokens` tokens
  mixed       the paper's long-context data mix: 60 % short and 40 % long sequences, lengths up to `longest`
  skewed      one sequence of half the tokens, then short ones (256 to 2048 tokens)
  ragged      few short sequences of any length, one-token and block-sized ones among them
and the budgets either from `topk` (blocks per query block) or from keep ratios drawn in keep_lo .. keep_hi (0 <= ratio
<= 1; `topk` 0 says so).  In a skewed batch the long sequence keeps keep_lo and the short ones 0.5 to 1.

Values are i.i.d. N(0, 1), as everywhere in this repository: routing scores are then close to random, kept blocks are
scattered over the whole past, and the gathers of K/V and Q/dO tiles meet the caches as rarely as they can.
"""
import random

import numpy as np
import torch

from paper_2604_13847_amd import binding as sb
from paper_2604_13847_amd import synth


def _case(kind, mix, tokens, hq, hkv, d, *, block=64, dtype="bf16", mode="per_qhead", topk=0, keep_lo=0.1, keep_hi=0.5, longest=16384, seed=0):
    return {"kind": kind, "mix": mix, "tokens": tokens, "hq": hq, "hkv": hkv, "d": d, "block": block, "dtype": dtype, "mode": mode,
            "topk": topk, "keep_lo": keep_lo, "keep_hi": keep_hi, "longest": longest, "batch_seed": seed}


def listed():
    cases = {
        # the smallest complete step: one short sequence, one head, float32 tensors (a unit of debugging and of gradient checks)
        "step_1k_one_head_f32": _case("step", "one", 1024, 1, 1, 64, dtype="f32", topk=4),
        # a short packed batch of ragged sequences, as at the end of an epoch or in fine-tuning on short samples
        "step_2k_ragged": _case("step", "ragged", 2039, 16, 2, 128, keep_lo=0.3, keep_hi=1.0),
        # the ordinary training step: a 32768-token pack, 32/8 heads, in both selection modes
        "step_32k": _case("step", "mixed", 32768, 32, 8, 128),
        "step_32k_per_kvgroup": _case("step", "mixed", 32768, 32, 8, 128, mode="per_kvgroup"),
        # a longer pack on seven query heads per KV head
        "step_64k_28_4": _case("step", "mixed", 65536, 28, 4, 128, keep_lo=0.05, keep_hi=0.3, longest=32768),
        # the paper's own setting, blocks of 256 tokens and 32 of them kept, on the head shapes of its two models
        "step_64k_block256": _case("step", "mixed", 65536, 16, 2, 128, block=256, topk=32, longest=32768),
        "step_64k_block256_d64": _case("step", "mixed", 65536, 14, 2, 64, block=256, topk=32, longest=32768),
        # one very long sequence at a fixed budget: gathers dominate
        "step_131k_top32": _case("step", "one", 131072, 32, 8, 128, topk=32),
        # the largest: one 131072-token sequence with many short ones behind it, 262144 tokens in all
        "step_262k_skewed": _case("step", "skewed", 262144, 32, 8, 128, keep_lo=0.05, keep_hi=0.05),
        # evaluation: forward only, odd token count
        "forward_40k": _case("forward", "mixed", 40001, 32, 8, 128, keep_lo=0.1, keep_hi=0.3),
        # the budget controller's part of a step on the longest sequence
        "controller_131k": _case("controller", "one", 131072, 32, 8, 128, topk=32),
        # a brought selection with an attention sink: few key blocks are kept by every query block
        "sink_64k": _case("sink", "one", 65536, 32, 8, 128, topk=24),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def draw(rng):
    """Another case of the same ranges, no dearer than the largest listed one."""
    most = 53e12  # operations of the largest listed case
    kind = rng.choice(["step", "step", "step", "forward", "controller", "sink"])
    lo, hi = {"step": (200, 200000), "forward": (200, 200000), "controller": (4000, 131072), "sink": (1000, 131072)}[kind]
    tokens = int(round(lo * (hi / lo) ** rng.random())) | (rng.random() < 0.5)
    hq, hkv = rng.choice([(32, 8), (32, 8), (28, 4), (16, 2), (14, 2), (4, 2), (8, 8), (1, 1)])
    d = rng.choice([128, 128, 64])
    block = rng.choice([64, 64, 64, 128, 256])
    mode = rng.choice(["per_qhead", "per_qhead", "per_kvgroup"])
    dtype = "f32" if tokens <= 16384 and rng.random() < 0.2 else "bf16"
    mix = rng.choice(["one", "mixed", "mixed", "skewed"]) if tokens > 8192 else rng.choice(["one", "ragged"])
    if kind in ("controller", "sink"):
        mix = "one"
    topk = rng.choice([0, 4, 16, 32, 64])
    if kind == "sink" and not topk:
        topk = 24
    keep_lo = rng.uniform(0.03, 0.3) if tokens > 8192 else rng.uniform(0.1, 1.0)
    c = _case(kind, mix, tokens, hq, hkv, d, block=block, dtype=dtype, mode=mode, topk=topk, keep_lo=keep_lo,
              keep_hi=keep_lo + (1.0 - keep_lo) * 0.4 * rng.random(), longest=max(2048, min(32768, tokens // 2)), seed=rng.randrange(1000))
    while work(c)["flops"] > most:  # a long sequence at a large keep ratio: halve the batch until it fits
        c["tokens"] //= 2
        c["longest"] = max(2048, c["longest"] // 2)
    return c


def _lengths(case):
    total, seed = case["tokens"], case["batch_seed"]
    if case["mix"] == "one":
        return [total]
    if case["mix"] == "mixed":
        top = case["longest"]
        return synth.mixed_lengths(seed, total, short=(top // 32, top // 4), long=(top // 2, top))
    rng = random.Random(seed)
    if case["mix"] == "skewed":
        lens, left = [total // 2], total - total // 2
        while left > 0:
            lens.append(min(left, rng.randint(256, 2048)))
            left -= lens[-1]
        return lens
    lens, left = [1, 64], total - 65
    while left > 0:
        lens.append(min(left, rng.randint(1, 700)))
        left -= lens[-1]
    return lens


def _batch(case):
    """(cu_seqlens, budgets) of the case's batch: the case alone decides them, the seed only draws values."""
    lens = _lengths(case)
    cu = synth.cu_from_lengths(lens)
    n = (np.diff(cu) + case["block"] - 1) // case["block"]
    if case["topk"]:
        return cu, np.full(len(lens), case["topk"], dtype=np.int32)
    rng = random.Random(case["batch_seed"] + 1)
    ratio = [rng.uniform(case["keep_lo"], case["keep_hi"]) for _ in lens]
    if case["mix"] == "skewed":
        ratio = [case["keep_lo"]] + [rng.uniform(0.5, 1.0) for _ in lens[1:]]
    return cu, np.clip(np.ceil(np.asarray(ratio) * n - 1e-6), 1, np.maximum(n, 1)).astype(np.int32)


def _problem(case, device):
    cu, topk = _batch(case)
    return sb.Problem(cu, topk, case["hq"], case["hkv"], case["d"], case["block"], dtype=sb.SB_F32 if case["dtype"] == "f32" else sb.SB_BF16,
                      select_mode=sb.SB_SELECT_PER_QHEAD if case["mode"] == "per_qhead" else sb.SB_SELECT_PER_KVGROUP, device=device)


def prepare(case, seed):
    dev = "cuda"
    pb = _problem(case, dev)
    lay, T = pb.layout, pb.T
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device=dev).manual_seed(seed)
    normal = lambda heads: torch.randn((T, heads, case["d"]), generator=gen, device=dev, dtype=dt)
    raw = lambda size: torch.empty(max(int(size), 256), dtype=torch.uint8, device=dev)
    st = {"kind": case["kind"], "pb": pb, "q": normal(case["hq"]), "k": normal(case["hkv"])}
    if case["kind"] != "sink":
        st["ws_scores"] = raw(lay.scores_ws_bytes)
    if case["kind"] == "controller":
        st.update(ws_cov=raw(lay.coverage_ws_bytes), ws_sel=raw(lay.select_ws_bytes))
        return st
    # what a training program allocates once: the plan, the workspaces and the outputs
    st.update(v=normal(case["hkv"]), plan=raw(lay.plan_bytes), ws_fwd=raw(lay.fwd_ws_bytes), o=torch.empty_like(st["q"]),
              lse=torch.empty((pb.Hq, T), dtype=torch.float32, device=dev))
    if case["kind"] != "forward":
        st.update(do=normal(case["hq"]), ws_bwd=raw(lay.bwd_ws_bytes), dq=torch.empty_like(st["q"]), dk=torch.empty_like(st["k"]),
                  dv=torch.empty_like(st["k"]))
    if case["kind"] == "sink":
        rowptr, idx = synth.sink_selection(pb.cu_host, case["block"], pb.topk_host, int(lay.sel_heads))
        st.update(rowptr=torch.from_numpy(rowptr).to(dev), idx=torch.from_numpy(idx).to(dev))
    return st


def run(st):
    pb, q, k = st["pb"], st["q"], st["k"]
    if st["kind"] == "controller":
        scores = sb.sb_block_scores(pb, q, k, ws=st["ws_scores"])
        coverage = sb.sb_score_coverage(pb, scores, ws=st["ws_cov"])
        rowptr, idx = sb.sb_select_topk(pb, scores, ws=st["ws_sel"])
        return scores, coverage, rowptr, idx
    if st["kind"] == "sink":
        rowptr, idx = st["rowptr"], st["idx"]
    else:
        _, rowptr, idx = sb.sb_score_select(pb, q, k, ws=st["ws_scores"], want_scores=st["kind"] == "step")
    sb.sb_plan_worklist(pb, rowptr, idx, plan=st["plan"])
    o, lse = sb.sb_sparse_attn_fwd(pb, q, k, st["v"], rowptr, idx, st["plan"], o=st["o"], lse=st["lse"], ws=st["ws_fwd"])
    if st["kind"] == "forward":
        return o, lse, rowptr, idx
    dq, dk, dv = sb.sb_sparse_attn_bwd(pb, q, k, st["v"], o, lse, st["do"], rowptr, idx, st["plan"], dq=st["dq"], dk=st["dk"], dv=st["dv"],
                                       ws=st["ws_bwd"])
    return (o, lse, dq, dk, dv) if st["kind"] == "sink" else (o, lse, dq, dk, dv, rowptr, idx)


def work(case):
    """Operations: 2 d per (past query block, key block) pair and selection head for the scores, 4 d per attended (query,
    key) pair and query head forward and 10 d backward, the diagonal block counted as its causal triangle.  Bytes: every
    tensor that goes in or comes out, once."""
    cu, topk = _batch(case)
    B, hq, hkv, d = case["block"], case["hq"], case["hkv"], case["d"]
    hs = hq if case["mode"] == "per_qhead" else hkv
    item = 4 if case["dtype"] == "f32" else 2
    pairs = past = entries = 0
    for L, k in zip(np.diff(cu).tolist(), topk.tolist()):
        n = -(-L // B)
        i = np.arange(n, dtype=np.int64)
        rows = np.minimum(B, L - i * B)
        c = np.minimum(min(k, n), i + 1)
        pairs += int(((c - 1) * rows * B + rows * (rows + 1) // 2).sum())
        past += n * (n - 1) // 2
        entries += int(c.sum())
    T, nblocks = int(cu[-1]), int((-(-np.diff(cu) // B)).sum())
    q_like, kv_like, lse = T * hq * d * item, T * hkv * d * item, 4 * T * hq
    selection = 4 * hs * (entries + nblocks)
    flops, size = 0, 0
    if case["kind"] != "sink":
        flops += 2 * d * past * hq
    if case["kind"] == "controller":
        # Q and K in; the scores of the past blocks, the curves and the selection out
        return {"flops": flops, "bytes": q_like + kv_like + 4 * hs * past + 4 * nblocks + selection}
    flops += 4 * d * pairs * hq
    size += q_like + 2 * kv_like + q_like + lse + selection          # Q, K, V; O, LSE; the selection
    if case["kind"] != "forward":
        flops += 10 * d * pairs * hq
        size += q_like + q_like + 2 * kv_like                        # dO; dQ, dK, dV
    return {"flops": flops, "bytes": size}


def tolerance(case):
    """About four times what was measured against float64 on small batches of the same kinds: bf16 outputs are off by up to
    2.4e-3 (2-norm) and 5.4e-2 (largest element), float32 scores and curves by 2e-7 and 2e-6.  Selected indices may differ
    where two scores tie within the rounding of a float32 sum."""
    if case["kind"] == "controller":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
    return {"rel": 1e-2, "max": 0.2, "differ": 1e-3}
