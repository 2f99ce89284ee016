"""Shared plumbing for the GPU parity tests: move seeded inputs to the device, run the library's
five calls through the Python binding, and run the CPU checker on the same inputs."""
import numpy as np
import torch

from oracle import oracle as orc
from paper_2604_13847_amd import binding as sb
from paper_2604_13847_amd import synth

DEV = "cuda:0"


def to_dev(x_f32: np.ndarray, dtype: str):
    if dtype == "bf16":
        return torch.from_numpy(synth.bf16_bits(x_f32)).to(DEV).view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(x_f32, dtype=np.float32)).to(DEV)


def to_host_f32(t: torch.Tensor) -> np.ndarray:
    return t.detach().float().cpu().numpy()


_last_tensors = [None, None]


def host_tensors(w: synth.Workload):
    """w.tensors(), keeping the most recent workload's arrays: the full-size tests run one workload in several
    selection modes, and drawing 2.7e9 normals takes longer than the GPU work."""
    key = (w.seed, tuple(w.lens), w.Hq, w.Hkv, w.D, w.dtype)
    if _last_tensors[0] != key:
        _last_tensors[0], _last_tensors[1] = None, None      # free the previous workload before drawing the next
        _last_tensors[1] = w.tensors()
        _last_tensors[0] = key
    return _last_tensors[1]


class Run:
    """One workload pushed through sb_block_scores -> sb_select_topk -> sb_plan_worklist -> fwd -> bwd."""

    def __init__(self, w: synth.Workload, mode: int, topk=None, do_bwd=True, sel_override=None):
        self.w, self.mode = w, mode
        t = host_tensors(w)
        self.host = t                                   # float32 arrays holding the storage-type values
        if topk is None:
            topk = w.topk if w.topk is not None else sb.sb_keep_ratio_to_topk(w.cu, w.B, w.keep_ratio)
        self.topk = np.asarray(topk, dtype=np.int32)
        dt = sb.SB_BF16 if w.dtype == "bf16" else sb.SB_F32
        self.pb = sb.Problem(w.cu, self.topk, w.Hq, w.Hkv, w.D, w.B, dtype=dt, select_mode=mode, device=DEV)
        self.opb = orc.Problem(w.cu, w.Hq, w.Hkv, w.D, w.B, mode)
        self.scale = 1.0 / np.sqrt(w.D)
        self.q, self.k, self.v, self.do = (to_dev(t[n], w.dtype) for n in ("q", "k", "v", "do"))
        self.scores = sb.sb_block_scores(self.pb, self.q, self.k)
        if sel_override is None:
            self.rowptr, self.idx = sb.sb_select_topk(self.pb, self.scores)
        else:
            self.rowptr = torch.from_numpy(np.ascontiguousarray(sel_override[0], dtype=np.int32)).to(DEV)
            self.idx = torch.from_numpy(np.ascontiguousarray(sel_override[1], dtype=np.int32)).to(DEV)
        self.plan = sb.sb_plan_worklist(self.pb, self.rowptr, self.idx)
        # every output starts as NaN: an element that no workgroup wrote stays NaN and fails all_written()
        nan = lambda like, shape=None: torch.full(shape or like.shape, float("nan"), dtype=like.dtype, device=DEV)
        self.o, self.lse = sb.sb_sparse_attn_fwd(self.pb, self.q, self.k, self.v, self.rowptr, self.idx, self.plan, o=nan(self.q),
                                                 lse=torch.full((w.Hq, w.T), float("nan"), dtype=torch.float32, device=DEV))
        if do_bwd:
            self.dq, self.dk, self.dv = sb.sb_sparse_attn_bwd(self.pb, self.q, self.k, self.v, self.o, self.lse, self.do,
                                                              self.rowptr, self.idx, self.plan, dq=nan(self.q), dk=nan(self.k),
                                                              dv=nan(self.k))
        torch.cuda.synchronize()
        self.all_written(do_bwd)
        self.rowptr_h = self.rowptr.cpu().numpy()
        self.idx_h = self.idx.cpu().numpy()[: int(self.rowptr_h[-1])]

    def all_written(self, bwd=True):
        """Every element of every output has been written with a number (holds at any size; the sampled comparisons of the
        full-size tests would not notice a work item that no workgroup took)."""
        names = ("o", "lse") + (("dq", "dk", "dv") if bwd else ())
        for n in names:
            t = getattr(self, n)
            assert bool(torch.isfinite(t).all()), f"{n}: elements left unwritten or not finite"

    def oracle_inputs(self):
        """What the checker sees: the storage values; float inputs are rounded to bf16 as the kernels do."""
        t = self.host
        if self.w.dtype == "bf16":
            return t["q"], t["k"], t["v"], t["do"]
        return tuple(synth.round_to_bf16(t[n]) for n in ("q", "k", "v", "do"))


# Tolerance: bf16 outputs against the float64 checker, max-abs 2e-2 and mean-abs 2e-3.
# An output stored as bf16 carries a rounding error of its own of up to half a unit in the last place, 2^-9 |x|
# (0.016 at |x| = 8, and dV reaches 7-8 on dense rows), which the absolute bound cannot see; so every element is held to
#     |got - ref| <= 2e-2 + 2^-8 |ref|
# (the literal bound plus one bf16 unit in the last place of the reference).  The same rounding has a mean: a quarter of a
# unit in the last place, between 2^-10 |x| and 2^-9 |x|; a tensor whose elements are all large (dV of a one-token
# sequence is the sum of its G query heads' dO: |x| = 1.8 on average for G = 5) exceeds 2e-3 by the store alone.  The mean
# of |got - ref| is therefore held to
#     2e-3 + 2^-10 mean|ref|
# i.e. the literal bound plus the least the bf16 store costs.  check_close also returns the literal max-abs error, which
# the tests print.
MAX_ABS, MEAN_ABS, ULP_BF16 = 2e-2, 2e-3, 2.0 ** -8
MEAN_ULP_BF16 = 2.0 ** -10
# LSE is stored in float32; the forward's row sum adds the probabilities as rounded to bf16 (the weights it applies to
# V), so it is off by at most 2^-9 relative, i.e. 2e-3 absolute in the logarithm; the rest is float32 arithmetic.
LSE_ABS = 4e-3


def err_stats(got: np.ndarray, ref: np.ndarray):
    """(worst |err| / (2e-2 + 2^-8 |ref|), mean |err|, literal max |err|)"""
    d = np.abs(got.astype(np.float64) - ref)
    if not d.size:
        return 0.0, 0.0, 0.0
    return float((d / (MAX_ABS + ULP_BF16 * np.abs(ref))).max()), float(d.mean()), float(d.max())


def check_close(name, got, ref):
    frac, mn, mx = err_stats(got, ref)
    assert np.isfinite(got).all(), f"{name}: non-finite values"
    mean_bound = MEAN_ABS + MEAN_ULP_BF16 * (float(np.abs(ref).mean()) if np.size(ref) else 0.0)
    assert frac <= 1.0 and mn <= mean_bound, (f"{name}: max-abs {mx:.4g} ({frac:.3f} of the bound 2e-2 + 2^-8|ref|) mean-abs {mn:.4g} "
                                             f"(ref max {np.abs(ref).max():.3g})")
    return round(mx, 5), round(mn, 6)


def check_lse(got, ref):
    d = float(np.abs(np.asarray(got, dtype=np.float64) - ref).max()) if np.size(ref) else 0.0
    assert d <= LSE_ABS, f"LSE: max-abs {d:.4g}"
    return round(d, 6)


def check_bwd_items(pv, colcost, nblk, qb_off, NQB, Hkv):
    """Key-major items: per KV head heaviest first; every column covered exactly once by one item or by parts with
    disjoint word ranges that span the column; only a column's last part may be lighter than the split weight."""
    items = pv["bwd_items"]
    wmax = pv["split_weight"]
    seq_of = np.repeat(np.arange(len(nblk)), nblk)
    parts = {}
    for g in range(Hkv):
        mine = items[g::Hkv]
        valid = mine[:, 0] >= 0
        nv = int(valid.sum())
        assert valid[:nv].all() and not valid[nv:].any()                      # the padding is at the end
        assert np.all(mine[:nv, 0] // NQB == g)
        assert np.all(np.diff(np.minimum(mine[:nv, 3], 4095)) <= 0)           # heaviest first
        for col, wr, slot, wt in mine[:nv]:
            parts.setdefault(int(col), []).append((int(wr) & 0xffff, int(wr) >> 16, int(slot), int(wt)))
    assert sorted(parts) == list(range(Hkv * NQB))                            # every column has an item
    split = {int(c): (int(s0), int(n)) for c, s0, n in pv["split_cols"]}
    slots = []
    for col, ps in parts.items():
        qb = col % NQB
        s = seq_of[qb]
        j, words = qb - int(qb_off[s]), (nblk[s] + 31) // 32
        ps.sort(key=lambda x: -x[0])                                          # part 0 covers the last query blocks
        assert ps[0][1] == words and ps[-1][0] == j // 32
        assert all(a[0] == b[1] for a, b in zip(ps[:-1], ps[1:]))             # contiguous, disjoint
        assert sum(x[3] for x in ps) == colcost[col]
        if len(ps) == 1:
            assert ps[0][2] == -1 and col not in split
        else:
            assert colcost[col] > wmax and all(x[3] >= wmax for x in ps[:-1])
            assert split[col] == (ps[0][2], len(ps)) and [x[2] for x in ps] == list(range(ps[0][2], ps[0][2] + len(ps)))
            slots += [x[2] for x in ps]
    assert sorted(slots) == list(range(pv["slots_used"])) and len(split) == len(pv["split_cols"])
    assert len(split) <= pv["split_max"] and len(slots) <= 2 * pv["split_max"]
    return len(split)
