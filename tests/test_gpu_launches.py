"""Launch shapes that depend on the size of the problem: each at the sizes where the rule changes, against the checker."""
import numpy as np
import pytest
import torch

from helpers import MAX_ABS, ULP_BF16, Run, check_close, check_lse, to_host_f32
from oracle import oracle as orc
from paper_2604_13847_amd import binding as sb
from paper_2604_13847_amd import synth
from test_gpu_parity import check_attention, check_plan, check_scores, check_selection, fused_selection_matches

pytestmark = pytest.mark.gpu


def check_backward_repeats(r, new_plan=False):
    """Two more backward calls into outputs and a workspace full of NaN: the same bits, whichever workgroup finishes first and
    whatever the workspace held."""
    first = {n: getattr(r, n).clone() for n in ("dq", "dk", "dv")}
    for _ in range(2):
        plan = sb.sb_plan_worklist(r.pb, r.rowptr, r.idx) if new_plan else r.plan
        again = {n: torch.full_like(x, float("nan")) for n, x in first.items()}
        ws = torch.full((max(int(r.pb.layout.bwd_ws_bytes), 256),), 0xff, dtype=torch.uint8, device="cuda")
        sb.sb_sparse_attn_bwd(r.pb, r.q, r.k, r.v, r.o, r.lse, r.do, r.rowptr, r.idx, plan, ws=ws, **again)
        torch.cuda.synchronize()
        for n, x in first.items():
            assert torch.equal(again[n].view(torch.uint8), x.view(torch.uint8)), n


# Key-major columns of a small problem are walked by several workgroups when the heaviest can have more than 16 tiles (twice
# the least run of 8): a column of the first block has (blocks * query heads per KV head) tiles at full budget.
@pytest.mark.parametrize("lens,Hq,Hkv,D,mode,ratio", [
    ([16 * 64], 1, 1, 64, 0, (1.0, 1.0)),                 # 16 tiles: one workgroup
    ([17 * 64 - 5], 1, 1, 64, 0, (1.0, 1.0)),             # 17 tiles: three workgroups, a ragged last block
    ([300, 64, 1, 577], 14, 2, 128, 0, (0.4, 1.0)),       # seven heads, ragged short sequences
    ([300, 64, 1, 577], 8, 2, 128, 1, (0.4, 1.0)),        # one selection for four heads
    ([2100], 16, 1, 64, 0, (1.0, 1.0)),                   # two rounds of eight selection heads: runs cross the rounds
    ([64 * 520 - 3], 2, 1, 64, 0, (0.01, 0.01)),          # runs cross the chunks of 256 query blocks (512 at D = 128)
    ([64 * 520 - 3], 2, 1, 128, 0, (0.01, 0.01)),
    ([64 * 257 - 3], 2, 1, 64, 0, (0.02, 0.02)),          # one query block past a chunk
    ([64 * 530 - 3], 2, 2, 64, 0, (0.02, 0.02)),          # 1060 columns: cut at head_dim 64 only, from half the weight on
])
def test_columns_of_small_problems_walked_by_several_workgroups(lens, Hq, Hkv, D, mode, ratio):
    w = synth.small_ragged(seed=71, lens=lens, Hq=Hq, Hkv=Hkv, D=D, ratio=ratio)
    r = Run(w, mode)
    print(w, check_attention(r), flush=True)
    check_backward_repeats(r, new_plan=True)  # the parts are added in walk order


# A column heavier than the split weight is cut into parts, and in a small problem a heavy part is itself walked by several
# workgroups: the reduction then adds, in walk order, the sums of whole parts and of parts' parts.  Block 0 is kept by every query
# block: 300 blocks with four heads (parts of 512, 512 and 176 tiles, all of them walked by several), 112 with seven heads on one KV
# head and on two (560 and 224), 545 with one (513 tiles for 16 workgroups and 32 for one); 128-token blocks have two such columns.
@pytest.mark.parametrize("blocks,B,Hq,Hkv,D,topk,mode", [
    (300, 64, 4, 1, 64, 4, 0), (300, 64, 4, 1, 128, 4, 0), (300, 64, 4, 1, 64, 4, 1), (300, 64, 4, 1, 128, 4, 1),
    (112, 64, 14, 2, 64, 8, 0), (112, 64, 7, 1, 64, 8, 1), (545, 64, 1, 1, 64, 31, 0), (545, 64, 1, 1, 128, 31, 0),
    (150, 128, 4, 1, 64, 4, 0),
])
def test_parts_of_split_columns_walked_by_several_workgroups(blocks, B, Hq, Hkv, D, topk, mode):
    w = synth.Workload("sink", [B * blocks - 9], Hq, Hkv, D, B=B, topk=[topk], seed=72)
    r = Run(w, mode, sel_override=synth.sink_selection(w.cu, B, w.topk, Hq if mode == 0 else Hkv))
    if B == 64:
        check_plan(r)
    pv = sb.plan_views(r.pb, r.plan)
    assert len(pv["split_cols"]) >= Hkv * (B // 64) and pv["sub_slots_used"] > len(pv["split_cols"])
    q, k, v, do = r.oracle_inputs()
    O, LSE = orc.attn_fwd(r.opb, q, k, v, r.rowptr_h, r.idx_h, r.scale)
    dQ, dK, dV = orc.attn_bwd(r.opb, q, k, v, do, r.rowptr_h, r.idx_h, r.scale)
    print(w, check_close("O", to_host_f32(r.o), O), check_lse(r.lse.cpu().numpy(), LSE), check_close("dQ", to_host_f32(r.dq), dQ))
    # the rows of a split column add up tens of thousands of rounded products: held to the size of the column instead of the element's
    heavy = np.zeros((w.T, Hkv), dtype=bool)
    for col in pv["split_cols"][:, 0]:
        g, tile = divmod(int(col), len(pv["qb_seq"]))
        at = slice(64 * tile, min(64 * tile + 64, w.T))
        heavy[at, g] = True
        for name, got, ref in (("dK", r.dk, dK), ("dV", r.dv, dV)):
            err = np.abs(to_host_f32(got[at, g]) - ref[at, g]).max()
            assert err <= MAX_ABS + ULP_BF16 * np.abs(ref[at, g]).max(), (name, col, err)
    for name, got, ref in (("dK", r.dk, dK), ("dV", r.dv, dV)):
        check_close(name, to_host_f32(got)[~heavy], ref[~heavy])
    check_backward_repeats(r, new_plan=True)


# Up to 64 sequences the kernels find their place by a scan across the lanes, from 65 on in tables in memory; the plan's work
# lists and its transpose are one launch for selection blocks of one tile and of several.
@pytest.mark.parametrize("S", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("B,mode", [(64, 0), (256, 1)])
def test_sequence_counts_around_a_wavefront(S, B, mode):
    lens = [[130, 1, 0, 64, 577][(7 * s) % 5] for s in range(S)]
    w = synth.small_ragged(seed=80 + S, lens=lens, Hq=4, Hkv=2, D=64, B=B, ratio=(0.3, 0.9))
    r = Run(w, mode)
    check_selection(r, check_scores(r))
    if B == 64:
        check_plan(r)
    fused_selection_matches(r)
    print(w, check_attention(r), flush=True)


class GrowingKeys(synth.Workload):
    """Keys grow along the sequence, so the softmax's reference point has to move again and again along a row."""

    def tensors(self):
        t = super().tensors()
        at = np.concatenate([np.arange(n) / max(n, 1) for n in self.lens])
        t["k"] = synth.round_to_bf16((t["k"] * (0.5 + 12.0 * at)[:, None, None]).astype(np.float32))
        return t


# The reference moves in a branch at head_dim 64 and in the kernel whose heads share tiles (three or four heads per KV head).
# O is an average of V with weights rounded to bf16 as their sum is: the bound of the other parity tests holds for any scores.
@pytest.mark.parametrize("Hq,Hkv,D,mode", [(2, 1, 64, 0), (4, 1, 64, 1), (3, 1, 128, 1), (4, 1, 128, 1), (2, 1, 128, 0)])
def test_reference_of_the_softmax_moves_along_the_row(Hq, Hkv, D, mode):
    lens = [1100, 65, 1, 64, 323]
    w = GrowingKeys("growing", lens, Hq, Hkv, D, keep_ratio=np.full(len(lens), 1.0), seed=90 + D + Hq)
    r = Run(w, mode, do_bwd=False)
    print(w, check_attention(r, bwd=False), flush=True)


# dQ of one query head per item at head_dim 128 is a software pipeline over a row's tiles, two tiles per iteration, with the block
# indices in a window of 64: rows of 1 to 5 tiles, of one less, as many and more than the window holds, and ragged ends in either
# 32-key half of the last tile.
@pytest.mark.parametrize("lens,Hq,Hkv,mode,dtype", [
    ([1, 33, 64, 65, 97, 128, 190, 256, 300], 2, 1, 0, "bf16"),
    ([1, 33, 64, 65, 97, 128, 190, 256, 300], 2, 2, 1, "bf16"),
    ([1, 33, 64, 65, 97, 128, 190, 256, 300], 1, 1, 0, "f32"),
    ([63 * 64, 64 * 64 - 40], 1, 1, 0, "bf16"),
    ([67 * 64 - 20], 1, 1, 0, "bf16"),
    ([133 * 64 - 1], 1, 1, 0, "bf16"),
])
def test_dq_of_one_head_per_item(lens, Hq, Hkv, mode, dtype):
    w = synth.small_ragged(seed=95, lens=lens, Hq=Hq, Hkv=Hkv, D=128, ratio=(1.0, 1.0), dtype=dtype)
    r = Run(w, mode)
    print(w, check_attention(r), flush=True)
    check_backward_repeats(r)


# The conversion of float32 inputs is one launch of at most 2^22 workgroups (2^32 elements); larger inputs are strided over.  Q, K and
# V together have 4.9e9 elements here, with values that bf16 holds, so the output is the bf16 call's before its rounding.
def test_float32_inputs_larger_than_one_launch():
    T, H, D = 200_000, 64, 128
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((T, H, D), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    n = (T + 63) // 64
    rowptr = torch.arange(H * n + 1, dtype=torch.int32, device="cuda")    # every query block keeps itself only
    idx = torch.arange(n, dtype=torch.int32, device="cuda").repeat(H)
    outs = []
    for dt in (sb.SB_BF16, sb.SB_F32):
        pb = sb.Problem([0, T], [1], H, H, D, dtype=dt, device="cuda")
        x = [t.float() if dt == sb.SB_F32 else t for t in (q, k, v)]
        nan = torch.full_like(x[0], float("nan"))
        outs.append(sb.sb_sparse_attn_fwd(pb, *x, rowptr, idx, sb.sb_plan_worklist(pb, rowptr, idx), o=nan))
        torch.cuda.synchronize()
        del x
    (o16, lse16), (o32, lse32) = outs
    assert torch.equal(o32.to(torch.bfloat16), o16) and torch.equal(lse32, lse16)
