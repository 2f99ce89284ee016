"""The query-major kernels at the edges of their pipelines: rows of one to a few tiles, the window of 64 block indices, ragged
last blocks, items of one and of two wavefronts, the ticketed tail of a launch, and scores that outgrow the softmax's reference.  Every
element against the float64 checker, with the tolerances of helpers.py."""
import numpy as np
import pytest
import torch

from helpers import Run, check_close, check_lse, to_host_f32
from oracle import oracle as orc
from paper_2604_13847_amd import binding as sb
from paper_2604_13847_amd import synth

pytestmark = pytest.mark.gpu

EDGES = (1, 31, 32, 33, 63, 64, 65, 96, 97, 128, 191, 257, 320, 385, 512, 575)


def check(w, mode, bwd=True):
    r = Run(w, mode, do_bwd=bwd)
    q, k, v, do = r.oracle_inputs()
    O, LSE = orc.attn_fwd(r.opb, q, k, v, r.rowptr_h, r.idx_h, r.scale)
    stats = {"O": check_close("O", to_host_f32(r.o), O), "LSE": check_lse(r.lse.cpu().numpy(), LSE)}
    if bwd:
        for name, got, ref in zip(("dQ", "dK", "dV"), (r.dq, r.dk, r.dv), orc.attn_bwd(r.opb, q, k, v, do, r.rowptr_h, r.idx_h, r.scale)):
            stats[name] = check_close(name, to_host_f32(got), ref)
    print(w, "mode", mode, stats, flush=True)
    return r


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode,Hq,Hkv,D", [(0, 2, 1, 128), (0, 24, 4, 128), (1, 4, 2, 128), (1, 40, 20, 128), (0, 2, 1, 64), (0, 48, 4, 64), (1, 6, 2, 64), (1, 48, 12, 64)])
def test_row_lengths_and_ragged_blocks(mode, Hq, Hkv, D, dtype):
    """Few items (two wavefronts each, four for dQ at head_dim 64) and many (one each): rows of 1 .. 9 tiles, sequences that end anywhere in
    a block."""
    w = synth.Workload("edges", EDGES, Hq, Hkv, D, keep_ratio=[1.0] * len(EDGES), dtype=dtype, seed=300 + Hq)
    check(w, mode)


@pytest.mark.parametrize("Hq,Hkv,D", [(2, 1, 128), (24, 8, 128), (32, 8, 64)])
def test_rows_longer_than_the_index_window(Hq, Hkv, D):
    w = synth.Workload("window", (64 * 70 - 5,), Hq, Hkv, D, topk=[67], seed=320 + Hq)
    check(w, 0, bwd=Hq != 24)


@pytest.mark.parametrize("lens,topk", [((64 * 300, 64 * 250 + 5), (3, 4)), ((64 * 80,) + (64 * 4,) * 120, (75,) + (2,) * 120)])
def test_ticketed_launches(lens, topk):
    """More than 4096 items of one wavefront each: all of them short, and those of one long sequence among short ones."""
    w = synth.Workload("tickets", lens, 8, 2, 128, topk=topk, seed=330 + len(lens))
    r = check(w, 0, bwd=len(lens) == 2)
    assert r.pb.layout.sel_rows >= 4096


# one sequence of 104 blocks at full budget and 4002 short ones: two wavefronts per item, tests/test_launch_variants.py holds it to them
LONG_AND_SHORT = ((64 * 104 - 3,) + (1, 40, 64) * 1334, (104,) + (1,) * 4002)


@pytest.mark.parametrize("D", [128, 64])
def test_ticketed_launches_of_two_wavefronts(D):
    """The ticket of an item passes from one wavefront to the other through LDS that strips are loaded into afterwards."""
    w = synth.Workload("tickets", LONG_AND_SHORT[0], 1, 1, D, topk=LONG_AND_SHORT[1], seed=335)
    r = check(w, 0)
    assert r.pb.layout.sel_rows >= 4096


JUMP = (64 * 9 + 17, 64 * 14, 40)
JUMP_SHAPES = {1: [(64, 16, 128), (192, 48, 64)], 2: [(2, 1, 128), (24, 8, 128), (24, 8, 64)]}  # wavefronts per item of the forward


@pytest.mark.parametrize("Hq,Hkv,D", JUMP_SHAPES[2] + JUMP_SHAPES[1])
@pytest.mark.parametrize("jump", [5.0, 13.0, 150.0])
def test_scores_that_outgrow_the_reference(Hq, Hkv, D, jump):
    """Scores that grow from block to block by `jump` powers of two and fall again: probabilities against the old reference are large or
    infinite, so the reference moves and what has been summed is rescaled; a row sees rises inside and across its tiles."""
    lens = JUMP
    w = synth.Workload("jump", lens, Hq, Hkv, D, topk=[12, 14, 1], seed=340 + Hq)
    t = w.tensors()
    u = np.full(D, D ** -0.5, dtype=np.float32)
    level = np.array([0, 1, 2, 3, 1, 0.5, 3, 0], dtype=np.float32) * jump / (8.0 * D ** -0.5 * 1.4427)
    for s, L in enumerate(lens):
        at = int(w.cu[s])
        steps = level[(np.arange(L) // 48) % len(level)]  # 48: rises also inside a 64-key tile and inside a 32-key strip
        t["k"][at:at + L] += (steps[:, None] * u)[:, None, :]
    t["q"] += 8.0 * u
    t = {n: synth.round_to_bf16(x) for n, x in t.items()}
    w.tensors = lambda: t
    w.seed = 1000 + w.seed + int(jump) + D  # (the arrays of a workload are kept by its seed)
    check(w, 0, bwd=False)


# Ten-, nine- and one-block sequences: few heads, two wavefronts per item; many, one (tests/test_launch_variants.py holds them to it).
# Four query heads per KV head: an element of dK and dV adds the roundings of every head's rows, sqrt(heads) times one head's, which with
# sixteen reaches 1.1 of the elementwise bound whatever the forward does.
SHORT = (64 * 9 + 17, 64 * 9, 40)
ONE_WAVEFRONT = [(0, 64, 16, 128), (0, 128, 32, 64)]
TWO_WAVEFRONTS = [(0, 4, 2, 128), (0, 4, 2, 64)]


@pytest.mark.parametrize("masked", [32, 64])
@pytest.mark.parametrize("mode,Hq,Hkv,D", ONE_WAVEFRONT + TWO_WAVEFRONTS + [(1, 8, 2, 128)])
def test_first_keys_that_score_minus_infinity(mode, Hq, Hkv, D, masked):
    """Channel 0 masks the first keys of every sequence: 16384 in the queries from the second block on times -1e35 in these keys is
    beyond float32, 0 in all others.  So the first strip or the first tile of those rows adds nothing, and the softmax's reference comes
    from a later one.  The channel's own gradients are sums of such numbers and are left out."""
    w = synth.Workload("masked", SHORT, Hq, Hkv, D, topk=[10, 9, 1], seed=350 + Hq + masked)
    t = w.tensors()
    for s, L in enumerate(SHORT):
        at = int(w.cu[s])
        t["q"][at:at + L, :, 0] = np.where(np.arange(L) < 64, 0.0, 16384.0)[:, None]
        t["k"][at:at + L, :, 0] = np.where(np.arange(L) < masked, -1e35, 0.0)[:, None]
    t = {n: synth.round_to_bf16(x) for n, x in t.items()}
    w.tensors = lambda: t
    w.seed += 2000 + D  # (the arrays of a workload are kept by its seed)
    r = Run(w, mode)
    q, k, v, do = r.oracle_inputs()
    O, LSE = orc.attn_fwd(r.opb, q, k, v, r.rowptr_h, r.idx_h, r.scale)
    stats = [check_close("O", to_host_f32(r.o), O), check_lse(r.lse.cpu().numpy(), LSE)]
    for name, got, ref in zip(("dQ", "dK", "dV"), (r.dq, r.dk, r.dv), orc.attn_bwd(r.opb, q, k, v, do, r.rowptr_h, r.idx_h, r.scale)):
        first = 0 if name == "dV" else 1
        stats.append(check_close(name, to_host_f32(got)[..., first:], ref[..., first:]))
    # the channel on in all queries: rows whose keys are all masked have no softmax, the others are what they were
    q = r.q.clone()
    q[:, :, 0] = 16384.0
    o, lse = sb.sb_sparse_attn_fwd(r.pb, q, r.k, r.v, r.rowptr, r.idx, r.plan)
    empty, same = np.zeros(w.T, dtype=bool), np.zeros(w.T, dtype=bool)
    for s, L in enumerate(SHORT):
        empty[w.cu[s]:w.cu[s] + min(L, masked)] = True
        same[w.cu[s] + min(L, 64):w.cu[s + 1]] = True
    assert bool(torch.isnan(o[empty]).all()) and not bool(torch.isfinite(lse[:, empty]).any())
    assert torch.equal(o[same], r.o[same]) and torch.equal(lse[:, same], r.lse[:, same])
    print(w, stats, flush=True)


@pytest.mark.parametrize("mode,Hq,Hkv,D", ONE_WAVEFRONT + TWO_WAVEFRONTS)
def test_an_infinite_value_stays_infinite(mode, Hq, Hkv, D):
    """One infinite element of V per sequence, in the first or the second 32-key strip: that column of O is infinite in every later block,
    everything else is what it is without it."""
    w = synth.Workload("infinite", SHORT, Hq, Hkv, D, topk=[10, 9, 1], seed=370 + Hq)
    r = Run(w, mode, do_bwd=False)
    for key, sign in ((3, 1.0), (40, -1.0)):
        v, want = r.v.clone(), r.o.clone()
        later = np.zeros(w.T, dtype=bool)
        for s, L in enumerate(SHORT[:2]):
            at = int(w.cu[s])
            v[at + key, :, 5] = sign * float("inf")
            want[at + 64:at + L, :, 5] = sign * float("inf")
            later[at + 64:at + L] = True
        o, lse = sb.sb_sparse_attn_fwd(r.pb, r.q, r.k, v, r.rowptr, r.idx, r.plan)
        assert torch.equal(o[later], want[later]) and torch.equal(lse, r.lse)


ROUNDED = (64,) * 8 + (128,) * 4 + (512,)


@pytest.mark.parametrize("mode,Hq,Hkv,D", ONE_WAVEFRONT)
def test_one_wavefront_rounds_no_more_than_two(mode, Hq, Hkv, D):
    """Float32 outputs, whose error is that of the probabilities' rounding to bf16: no larger than with a reference of its own for the even
    and for the odd 32-key strips of a row, whose largest scores of the first strip are then exact, as two wavefronts have it."""
    w = synth.Workload("rounded", ROUNDED, Hq, Hkv, D, keep_ratio=[1.0] * len(ROUNDED), dtype="f32", seed=360 + Hq)
    r = Run(w, mode, do_bwd=False)
    q, k, v, _ = r.oracle_inputs()
    O, _ = orc.attn_fwd(r.opb, q, k, v, r.rowptr_h, r.idx_h, r.scale)
    heads = range(0, Hq, Hq // 8)
    for lo, hi in ((0, 512), (512, 1024), (1024, 1536)):  # rows of one tile, of up to two, of up to eight
        two = here = 0.0
        for s in range(len(ROUNDED)):
            at = slice(int(w.cu[s]), int(w.cu[s + 1]))
            if not lo <= at.start < hi:
                continue
            n = np.arange(at.stop - at.start)
            for h in heads:
                g = h * Hkv // Hq
                x = q[at, h].astype(np.float64) @ k[at, g].astype(np.float64).T * r.scale
                x[n[:, None] < n] = -np.inf
                num, den = 0.0, 0.0
                top = x.max(axis=1)
                for odd in (0, 1):
                    mine = n // 32 % 2 == odd
                    m = x[:, mine][:, :32].max(axis=1)
                    seen = np.isfinite(m)
                    p = np.exp(np.where(seen[:, None], x[:, mine] - np.where(seen, m, 0.0)[:, None], -np.inf))
                    p = synth.round_to_bf16(p.astype(np.float32)).astype(np.float64) * np.exp(np.where(seen, m, 0.0) - top)[:, None]
                    num, den = num + p @ v[at, g][mine].astype(np.float64), den + p.sum(axis=1)
                two += ((num / den[:, None] - O[at, h]) ** 2).sum()
                here += ((to_host_f32(r.o[at, h]) - O[at, h]) ** 2).sum()
        print(w, (lo, hi), "two references", two ** 0.5, "here", here ** 0.5, flush=True)
        assert here <= two
