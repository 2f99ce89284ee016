"""Forms that small problems take: scores and selection by one kernel that writes the matrix too, plans of two launches, and the walk of
key-major columns of few tiles; and the histogram sort of the coverage curves.  Sizes lie at the edges of each rule."""
import ctypes as C

import numpy as np
import pytest
import torch

from helpers import DEV, Run
from oracle import dst_oracle as dst
from oracle import oracle as orc
from paper_2604_13847_amd import binding as sb
from paper_2604_13847_amd import synth
from test_gpu_parity import check_attention, check_plan

pytestmark = pytest.mark.gpu


# (lens, Hq, Hkv, D, mode), by one kernel: up to 256 workgroups (16 blocks and a selection head each) and 448 blocks a sequence, whose keys fit the
# LDS (tests/test_launch_variants.py); from 257 blocks on a wavefront computes more than one tile, 65 sequences read tables instead of lanes
AT_ONCE = [((64 * 447 + 1,), 8, 8, 128, 0, True), ((64 * 448 + 1,), 8, 8, 128, 0, False), ((64 * 300,), 8, 2, 64, 1, True), ((64 * 256,), 16, 2, 128, 0, True),
           ((64 * 257,), 16, 2, 128, 0, False), ((64 * 128,), 32, 8, 64, 0, True), ((64 * 128, 1), 32, 8, 64, 0, False), ((1,), 1, 1, 64, 0, True),
           ((64, 1, 0, 65) * 9, 6, 2, 64, 1, True), ((1, 63, 700) * 22, 4, 2, 128, 1, True), ((64 * 16, 64 * 15 + 1, 64 * 17 - 1), 4, 4, 64, 0, True),
           ((100,) * 40, 16, 2, 128, 0, True)]


@pytest.mark.parametrize("lens,Hq,Hkv,D,mode", [a[:5] for a in AT_ONCE])
def test_scores_and_selection_at_once(lens, Hq, Hkv, D, mode):
    """The same bits as sb_block_scores and sb_select_topk, -infinity included, in buffers that held NaN and -1."""
    w = synth.small_ragged(seed=500 + Hq, lens=lens, Hq=Hq, Hkv=Hkv, D=D, ratio=(0.1, 0.9))
    r = Run(w, mode, do_bwd=False)
    lay, nnz = r.pb.layout, int(r.rowptr_h[-1])
    scores = torch.full((lay.scores_elems,), float("nan"), device=DEV)
    rowptr, idx = (torch.full((n,), -1, dtype=torch.int32, device=DEV) for n in (lay.sel_rows + 1, lay.sel_nnz))
    ws = torch.empty(lay.scores_ws_bytes, dtype=torch.uint8, device=DEV)
    ptr = lambda x: C.c_void_p(x.data_ptr()) if x is not None else None
    rc = sb.lib().sb_score_select(r.pb.ref(), *map(ptr, (r.q, r.k, None, scores, rowptr, idx, ws)), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, sb.lib().sb_last_error().decode()
    torch.cuda.synchronize()
    assert torch.equal(scores.view(torch.int32), r.scores[: lay.scores_elems].view(torch.int32))
    assert torch.equal(rowptr, r.rowptr) and torch.equal(idx[:nnz], r.idx[:nnz])


# (lens, Hq, Hkv, mode), in two launches: up to 512 blocks, 64 sequences and 4096 bitmap words of a KV head's columns (tests/test_launch_variants.py)
PLANS = [((64 * 127 + 1,), 8, 1, 0, True), ((64 * 128 + 1,), 8, 1, 0, False), ((64 * 256,), 4, 2, 0, True), ((64 * 257,), 4, 2, 0, False),
         ((64 * 363,), 2, 2, 1, False), ((64 * 341,), 2, 2, 1, True), ((64 * 20,) * 25 + (64 * 12,), 4, 2, 0, True), ((64 * 20,) * 25 + (64 * 13,), 4, 2, 0, False),
         ((0, 1, 0, 130) * 16, 4, 2, 1, True), ((0, 1, 0, 130, 0) * 13, 4, 2, 1, False), ((700, 64 * 40, 1, 64 * 9), 8, 2, 0, True), ((2039,), 16, 2, 0, True),
         ((1,), 1, 1, 1, True)]


@pytest.mark.parametrize("lens,Hq,Hkv,mode", [p[:4] for p in PLANS])
def test_plans_of_two_launches(lens, Hq, Hkv, mode):
    w = synth.small_ragged(seed=520 + Hq, lens=lens, Hq=Hq, Hkv=Hkv, D=64, ratio=(0.05, 0.2))
    r = Run(w, mode)
    check_plan(r)
    if w.T <= 4096:
        print(w, check_attention(r), flush=True)


@pytest.mark.parametrize("lens,Hq,Hkv,mode", [p[:4] for p in PLANS if p[0][0] >= 64 * 127 or p[0][0] == 700])
def test_plans_of_two_launches_with_a_sink(lens, Hq, Hkv, mode):
    """Every row keeps block 0: its column is cut where it has more than 512 tiles, and walked by several workgroups, so that entries of both
    lists are used and others are not."""
    w = synth.Workload("sink", list(lens), Hq, Hkv, 64, topk=[3] * len(lens), seed=525 + Hq)
    r = Run(w, mode, sel_override=synth.sink_selection(w.cu, 64, w.topk, Hq if mode == 0 else Hkv))
    check_plan(r)
    pv = sb.plan_views(r.pb, r.plan)
    if Hkv * r.pb.layout.num_qblocks < 1024:  # (more columns fill the chip uncut)
        assert pv["sub_slots_used"] > 0
    # (cut where the tiles of its words of 32 rows but the first are 512 and more)
    assert (len(pv["split_cols"]) > 0) == (Hq // Hkv * (-(-max(lens) // 64) - 32) >= 512)
    items = pv["bwd_items"][:, 0]
    assert 0 < (items >= 0).sum() <= len(items)


def test_plan_in_a_buffer_that_held_another():
    """Nothing that an earlier plan, or anything else, left in the buffer shows: unused entries are written in every call."""
    w = synth.small_ragged(seed=530, lens=(64 * 37 - 9, 200), Hq=8, Hkv=2, D=128, ratio=(0.6, 0.9))
    r = Run(w, 0)
    for fill in (0, 0x7f, 0xff):
        plan = torch.full_like(r.plan, fill)
        sb.sb_plan_worklist(r.pb, r.rowptr, r.idx, plan=plan)
        grads = sb.sb_sparse_attn_bwd(r.pb, r.q, r.k, r.v, r.o, r.lse, r.do, r.rowptr, r.idx, plan)
        torch.cuda.synchronize()
        r.plan = plan
        check_plan(r)
        for a, b in zip(grads, (r.dq, r.dk, r.dv)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,mode", [(1, 1, 0), (3, 1, 0), (2, 1, 1), (9, 1, 0)])
def test_columns_of_few_tiles(Hq, Hkv, mode, D):
    """One to some twenty tiles a column, odd and even, with one to nine of them on the diagonal, none of them or all of them."""
    lens = [64 * n - 17 * (n % 3) for n in range(1, 8)] + [1, 33]
    w = synth.Workload("few", lens, Hq, Hkv, D, topk=[1, 2, 2, 3, 3, 7, 2, 1, 1], seed=540 + Hq)
    print(check_attention(Run(w, mode)), flush=True)


KINDS = {
    "normal": lambda rng, s: rng.normal(size=s),
    "wide": lambda rng, s: rng.normal(size=s) * 40.0,
    "equal": lambda rng, s: np.full(s, 1.5),
    "few values": lambda rng, s: rng.integers(0, 40, size=s) * 0.25,          # bins of 32 keys and more
    "thirty to a value": lambda rng, s: np.argsort(rng.random(s), axis=-1) // 30 * 0.01,  # just below
    "outlier": lambda rng, s: rng.normal(size=s) + 1e4 * (rng.random(s) < 1.0 / s[-1]),
    "masked": lambda rng, s: np.where(rng.random(s) < 0.01, -np.inf, rng.normal(size=s)),
    "half masked": lambda rng, s: np.where(rng.random(s) < 0.5, -np.inf, rng.normal(size=s)),
    "tiny": lambda rng, s: rng.normal(size=s) * 1e-30,
    "not a number": lambda rng, s: np.where(rng.random(s) < 0.01, np.nan, rng.normal(size=s)),  # counts as -infinity
}


def check_curves(sc):
    """sc: [heads][n][n].  The curves against the float64 checker (2e-6, as in tests/test_gpu_dst.py: shares are at most 1 and a curve is a
    mean of row sums)."""
    Hs, n = sc.shape[:2]
    cu = np.array([0, n * 64 - 5])
    pb = sb.Problem(cu, [8], Hs, Hs, 64, 64, device=DEV)
    po = orc.Problem(cu, Hs, Hs, 64, 64, 0)
    got = sb.sb_score_coverage(pb, torch.from_numpy(sc.ravel()).to(DEV)).cpu().numpy()[:n]
    with np.errstate(invalid="ignore"):
        ref = dst.coverage_curves(po.nblk, po.Hs, np.where(np.isnan(sc), -np.inf, sc).ravel(), po.score_off)
    np.testing.assert_allclose(got, ref, rtol=0, atol=2e-6)  # (NaN where the checker has NaN)
    return ref


# 1025 blocks are the most of the kernel that ends with 16 keys a lane, 2049 of the one with 32
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("n", [300, 1025, 1026, 2049])
def test_coverage_sorted_by_a_histogram(kind, n):
    """Rows of 257 to 2048 keys: spread, tied, with outliers that leave all others in one bin, and with -infinity and NaN among them."""
    Hs = 2
    sc = KINDS[kind](np.random.default_rng(n), (Hs, n, n)).astype(np.float32)
    sc[:, :, 0] = np.where(np.isfinite(sc[:, :, 0]), sc[:, :, 0], 0.0)  # (a row without any finite score has no softmax)
    check_curves(sc)


# up to 64 sequences the kernel of the rows writes the tables that the column sums read, beyond them a kernel before it
@pytest.mark.parametrize("lens", [(0, 700, 0, 1), (64 * 300, 0, 0), (0, 130, 64) * 21 + (0,), (0, 130, 64) * 22])
def test_coverage_of_packs_with_empty_sequences(lens):
    rng, cu = np.random.default_rng(7), np.concatenate([[0], np.cumsum(lens)])
    po = orc.Problem(cu, 2, 1, 64, 64, 0)
    sc = rng.normal(size=sum(2 * n * n for n in po.nblk)).astype(np.float32)
    pb = sb.Problem(cu, [8] * len(lens), 2, 1, 64, 64, device=DEV)
    ws = torch.full((pb.layout.coverage_ws_bytes,), 0x7f, dtype=torch.uint8, device=DEV)
    got = sb.sb_score_coverage(pb, torch.from_numpy(sc).to(DEV), ws=ws).cpu().numpy()[: po.NQB]
    assert np.abs(got - dst.coverage_curves(po.nblk, 2, sc, po.score_off)).max() <= 2e-6


@pytest.mark.parametrize("Hs", [1, 3, 5, 11, 40])
def test_coverage_of_heads_that_differ(Hs):
    """Groups of one to ten heads, of which a wavefront sorts up to three in turn (of 5, the last group has none): rows that the histogram
    sorts and rows that it leaves to the network, in any order, on the same LDS."""
    rng, n = np.random.default_rng(6), 300
    sc = rng.normal(size=(Hs, n, n)).astype(np.float32)
    tied = rng.random((Hs, n)) < 0.3
    sc[tied] = np.round(sc[tied])
    check_curves(sc)


def test_coverage_of_rows_without_a_softmax():
    """One row with +infinity and one without a finite key, each left to the network: NaN for the budgets that they count for (up to
    their 271 and 281 blocks), as the definition gives it, and nothing else is touched."""
    n = 700
    sc = np.random.default_rng(5).normal(size=(2, n, n)).astype(np.float32)
    sc[0, 270, :270] = -np.inf
    sc[1, 280, 17] = np.inf
    ref = check_curves(sc)
    assert np.isnan(ref[1:280]).all() and np.isfinite(ref[280:]).all()


@pytest.mark.parametrize("n", [257, 513, 1025, 2049, 2050])
@pytest.mark.parametrize("k", [2, 40, 0.6])
def test_selection_of_rows_in_registers(n, k):
    """Rows on both sides of every register count and of the form that keeps its keys in LDS (2050 blocks), budgets on both sides of the
    switch between the two threshold searches; ties, NaN, -infinity and signed zeros among the scores.  Bit for bit the checker's order."""
    budget = k if isinstance(k, int) else int(k * n)
    rng = np.random.default_rng(n + budget)
    sc = rng.normal(size=(1, n, n)).astype(np.float32)
    sc[:, 1::3] = np.round(sc[:, 1::3] * 4.0) / 4.0
    sc[rng.random(sc.shape) < 0.02] = np.nan
    sc[rng.random(sc.shape) < 0.02] = -np.inf
    sc[rng.random(sc.shape) < 0.02] = -0.0
    cu = np.array([0, n * 64 - 63])
    pb = sb.Problem(cu, [budget], 1, 1, 64, 64, device=DEV)
    rowptr, idx = sb.sb_select_topk(pb, torch.from_numpy(sc.ravel()).to(DEV))
    rp, ix = orc.select_topk(orc.Problem(cu, 1, 1, 64, 64, 0), sc.ravel(), np.array([budget], dtype=np.int32))
    assert np.array_equal(rowptr.cpu().numpy(), rp) and np.array_equal(idx.cpu().numpy()[: int(rp[-1])], ix)
