"""Lists that are handed out by ticket: query-major launches that hold items back, and the key-major launch, whose
last columns are drawn (tests/test_gpu_deals.py has every form).  Every element against the float64 checker, so that an item that nobody drew shows, and the same bits from a
second run, whoever draws what."""
import numpy as np
import pytest
import torch

from helpers import Run, check_close, check_lse, to_host_f32
from oracle import oracle as orc
from paper_2604_13847_amd import binding as sb
from paper_2604_13847_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,Hq,Hkv,D,blocks", [(0, 8, 8, 128, 531), (1, 16, 8, 64, 531), (1, 18, 9, 128, 467)])
def test_columns_and_items_by_ticket(mode, Hq, Hkv, D, blocks):
    """More than 4096 items and columns of a selection with a sink: block 0's column is cut where it has more than 512 tiles, so that KV
    heads' lists end with entries that are none; nine selection heads of 467 blocks are no multiple of 8, so that a few ids have no item.
    dK and dV of block 0 add the roundings of all rows and are held to the block's largest element (tests/test_gpu_parity.py has the
    reason), everything else to the tolerances of helpers.py."""
    w = synth.Workload("tickets", (64 * blocks - 59,), Hq, Hkv, D, topk=[2], seed=390 + Hq)
    r = Run(w, mode, sel_override=synth.sink_selection(w.cu, 64, w.topk, Hq if mode == 0 else Hkv))
    assert r.pb.layout.sel_rows >= 4096 and Hkv * blocks >= 4096
    q, k, v, do = r.oracle_inputs()
    O, LSE = orc.attn_fwd(r.opb, q, k, v, r.rowptr_h, r.idx_h, r.scale)
    dQ, dK, dV = orc.attn_bwd(r.opb, q, k, v, do, r.rowptr_h, r.idx_h, r.scale)
    stats = [check_close("O", to_host_f32(r.o), O), check_lse(r.lse.cpu().numpy(), LSE), check_close("dQ", to_host_f32(r.dq), dQ)]
    for name, got, ref in (("dK", to_host_f32(r.dk), dK), ("dV", to_host_f32(r.dv), dV)):
        stats.append(check_close(name, got[64:], ref[64:]))
        most = np.abs(ref[:64]).max(axis=(0, 2))
        assert (np.abs(got[:64] - ref[:64]).max(axis=(0, 2)) <= 2e-2 + 2.0 ** -8 * most).all()
    print(w, "mode", mode, stats, flush=True)
    o, lse = sb.sb_sparse_attn_fwd(r.pb, r.q, r.k, r.v, r.rowptr, r.idx, r.plan)
    grads = sb.sb_sparse_attn_bwd(r.pb, r.q, r.k, r.v, r.o, r.lse, r.do, r.rowptr, r.idx, r.plan)
    torch.cuda.synchronize()
    for a, b in ((o, r.o), (lse, r.lse), *zip(grads, (r.dq, r.dk, r.dv))):
        assert torch.equal(a, b)
