"""Every way in which a launch hands its items out: by position, one in sixteen held back, the last quarter drawn, drawn one after the other;
key-major columns by position and drawn.  tests/test_launch_variants.py holds the shapes to the form they mean.  Each element against plain
float32 torch, head by head, so that an item that nobody took, or two did, shows, and the same bits from a second run."""
import numpy as np
import pytest
import torch

from helpers import DEV, check_close, check_lse
from paper_2604_13847_amd import binding as sb

pytestmark = pytest.mark.gpu

# (mode, Hq, Hkv, D, blocks, budget), forward's and dQ's form, columns drawn; the sequence is 59 tokens short of its blocks
SHAPES = [
    ((0, 8, 8, 128, 531, 2), "position", "held", True), ((0, 8, 8, 128, 531, 16), "draw", "held", True), ((0, 8, 8, 128, 531, 26), "draw", "draw", True),
    ((0, 16, 16, 64, 531, 4), "position", "held", False), ((0, 8, 8, 64, 531, 34), "last", "last", True),
    # seven query heads of a KV head: ids in groups of 56, with none for some of the last
    ((1, 63, 9, 64, 467, 3), "position", "held", False), ((1, 63, 9, 64, 467, 13), "last", "held", True), ((1, 63, 9, 128, 467, 2), "position", "draw", True),
    # heads that share a workgroup, in one plane and in two
    ((1, 36, 9, 128, 467, 3), "group", "draw", True), ((1, 72, 9, 128, 467, 2), "group", "draw", True),
]


def reference(pb, L, h, hs, g, q, k, v, do, rowptr, idx):
    """(O, LSE, dQ, dK, dV) of query head h, which keeps selection head hs's blocks of KV head g"""
    n, D, c = (L + 63) // 64, pb.D, int(pb.topk_host[0])
    tiles = lambda x: torch.nn.functional.pad(x.float(), (0, 0, 0, 64 * n - L)).reshape(n, 64, D)
    Q, K, V, dO = tiles(q[:, h]), tiles(k[:, g]), tiles(v[:, g]), tiles(do[:, h])
    row = rowptr[hs * n: hs * n + n + 1].long()
    at = row[:n, None] + torch.arange(c, device=DEV)
    kept = at < row[1:, None]
    j = torch.where(kept, idx[at.clamp(max=idx.numel() - 1)].long(), 0)
    for x in (Q, K, V):
        x.requires_grad_()
    KK, VV = K[j].reshape(n, c * 64, D), V[j].reshape(n, c * 64, D)
    key = (64 * j[:, :, None] + torch.arange(64, device=DEV)).reshape(n, 1, c * 64)
    query = (64 * torch.arange(n, device=DEV)[:, None] + torch.arange(64, device=DEV))[:, :, None]
    open_ = (key <= query) & kept.repeat_interleave(64, 1)[:, None]
    S = torch.where(open_, torch.bmm(Q, KK.transpose(1, 2).contiguous()) / D ** 0.5, -torch.inf)
    O = torch.bmm(torch.softmax(S, -1), VV)
    O.backward(dO)
    flat = lambda x: x.detach().reshape(64 * n, D)[:L]
    return flat(O), torch.logsumexp(S, -1).detach().reshape(-1)[:L], flat(Q.grad), flat(K.grad), flat(V.grad)


@pytest.mark.parametrize("shape", [s[0] for s in SHAPES])
def test_every_form_takes_every_item_once(shape):
    mode, Hq, Hkv, D, blocks, budget = shape
    L = 64 * blocks - 59
    gen = torch.Generator(device=DEV).manual_seed(sum(shape))
    q, k, v, do = (torch.randn((L, heads, D), generator=gen, device=DEV, dtype=torch.bfloat16) for heads in (Hq, Hkv, Hkv, Hq))
    pb = sb.Problem([0, L], [budget], Hq, Hkv, D, select_mode=mode, device=DEV)
    _, rowptr, idx = sb.sb_score_select(pb, q, k)
    plan = sb.sb_plan_worklist(pb, rowptr, idx)
    nan = lambda x: torch.full_like(x, float("nan"))

    def step():
        lse = torch.full((Hq, L), float("nan"), device=DEV)
        o, lse = sb.sb_sparse_attn_fwd(pb, q, k, v, rowptr, idx, plan, o=nan(q), lse=lse)
        return (o, lse) + tuple(sb.sb_sparse_attn_bwd(pb, q, k, v, o, lse, do, rowptr, idx, plan, dq=nan(q), dk=nan(k), dv=nan(k)))

    first, second = step(), step()
    torch.cuda.synchronize()
    for a, b in zip(first, second):
        assert torch.equal(a, b)
    o, lse, dq, dk, dv = first
    host = lambda x: x.float().cpu().numpy()
    G, worst = Hq // Hkv, {}
    for g in range(Hkv):
        dK = dV = 0.0
        for h in range(g * G, (g + 1) * G):
            O, LSE, dQ, dk_h, dv_h = reference(pb, L, h, h if mode == 0 else g, g, q, k, v, do, rowptr, idx)
            dK, dV = dK + dk_h, dV + dv_h
            check_lse(host(lse[h]), host(LSE).astype(np.float64))
            for name, got, ref in (("O", o[:, h], O), ("dQ", dq[:, h], dQ)):
                worst[name] = max(worst.get(name, 0.0), check_close(name, host(got), host(ref).astype(np.float64))[0])
        for name, got, ref in (("dK", dk[:, g], dK), ("dV", dv[:, g], dV)):
            worst[name] = max(worst.get(name, 0.0), check_close(name, host(got), host(ref).astype(np.float64))[0])
    print(shape, worst, flush=True)
