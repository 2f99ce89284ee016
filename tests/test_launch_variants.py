"""Which form of a kernel a problem takes is decided by its sizes.  The tests on the GPU that mean one form by their shapes are held to
it here, in a process whose HIP launch calls only write down what would be launched (CPU only; no buffer is read)."""
import json
import os
import re
import subprocess
import sys

import pytest

import test_gpu_deals as deals
import test_gpu_head_rows as rows
import test_gpu_small_plans as small

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CALLS = """
import ctypes as C, json, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
shim.recorded_kernel.restype = C.c_char_p
import numpy as np
from paper_2604_13847_amd import binding as sb
lens, topk, mode, Hq, Hkv, D = json.loads(sys.argv[2])
pb = sb.Problem(np.concatenate([[0], np.cumsum(lens)]), topk, Hq, Hkv, D, select_mode=mode)
pb.c.cu_seqlens_dev = pb.c.topk_dev = 4096
b, lib, p = C.c_void_p(4096), sb.lib(), pb.ref()
sb._check(lib.sb_sparse_attn_fwd(p, b, b, b, b, b, b, b, b, b, None))
sb._check(lib.sb_sparse_attn_bwd(p, b, b, b, b, b, b, b, b, b, b, b, b, b, None))
if len(sys.argv) > 3:  # the plan, and scores with a selection
    sb._check(lib.sb_plan_worklist(p, b, b, b, None))
    sb._check(lib.sb_score_select(p, b, b, None, b, b, b, b, None))
out = np.zeros((256, 6), dtype=np.uint32)
for i in range(shim.recorded_launches(out.ctypes.data_as(C.c_void_p))):
    print("kernel", shim.recorded_kernel(i).decode(), out[i][0])
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """(lens, topk, mode, Hq, Hkv, D) -> [(kernel, workgroups)] of a forward and a backward, and of plan and selection if asked for"""
    shim = str(tmp_path_factory.mktemp("launch") / "record_launches.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(ROOT, "tests", "launch", "record_launches.c")], check=True)

    def of(*problem, before=()):
        r = subprocess.run([sys.executable, "-c", CALLS, shim, json.dumps(problem), *before], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout[-3000:]
        return [(l.split()[1], int(l.split()[2])) for l in r.stdout.splitlines() if l.startswith("kernel ")]

    return of


@pytest.fixture(scope="module")
def query_major(launches):
    """(lens, topk, mode, Hq, Hkv, D) -> wavefronts per item of the forward and of dQ (4: the kernel for few items) and whether items
    are handed out by ticket."""
    def of(*problem):
        names = [name for name, _ in launches(*problem)]
        fwd = [m[1] for n in names if (m := re.search(r"attn_fwd_head_kernelILi\d+ELb[01]ELi(\d)E", n))]
        dq = [m[1] for n in names if (m := re.search(r"attn_bwd_dq_head_kernelILi\d+ELb[01]ELi(\d)E", n))] + ["4" for n in names if "attn_bwd_dq_kernel" in n]
        assert len(fwd) == len(dq) == 1, names
        return int(fwd[0]), int(dq[0]), any("fill" in n for n in names)

    return of


@pytest.mark.parametrize("shape", rows.ONE_WAVEFRONT + rows.TWO_WAVEFRONTS)
def test_short_sequences(query_major, shape):
    fwd, dq, _ = query_major(rows.SHORT, [10, 9, 1], *shape)
    assert (fwd, dq) == ((1, 1) if shape in rows.ONE_WAVEFRONT else (2, 2 if shape[3] == 128 else 4))


@pytest.mark.parametrize("shape", rows.ONE_WAVEFRONT)
def test_rounding(query_major, shape):
    budgets = [(L + 63) // 64 for L in rows.ROUNDED]
    assert query_major(rows.ROUNDED, budgets, *shape)[0] == 1


@pytest.mark.parametrize("wavefronts,shape", [(n, s) for n, shapes in rows.JUMP_SHAPES.items() for s in shapes])
def test_moving_reference(query_major, wavefronts, shape):
    assert query_major(rows.JUMP, [12, 14, 1], 0, *shape)[0] == wavefronts


@pytest.mark.parametrize("D", [128, 64])
def test_tickets_of_two_wavefronts(query_major, D):
    assert query_major(*rows.LONG_AND_SHORT, 0, 1, 1, D) == (2, 2, True)


@pytest.mark.parametrize("lens,topk", [((64 * 300, 64 * 250 + 5), (3, 4)), ((64 * 80,) + (64 * 4,) * 120, (75,) + (2,) * 120)])
def test_tickets_of_one_wavefront(query_major, lens, topk):
    assert query_major(lens, topk, 0, 8, 2, 128) == (1, 1, True)


@pytest.mark.parametrize("shape,forward,dq,columns", deals.SHAPES)
def test_how_items_are_handed_out(launches, shape, forward, dq, columns):
    mode, Hq, Hkv, D, blocks, budget = shape
    heads = 1 if mode == 0 else Hq // Hkv
    items = blocks * (Hq if mode == 0 else Hkv)
    ids = (items + 7) // 8 * 8 * heads
    of_grid = {(ids + 7) // 8 * 8: "position", (ids + ids // 128 * 8 + 7) // 8 * 8: "held", (ids + ids // 64 + 7) // 8 * 8: "last"}
    made = launches((64 * blocks - 59,), (budget,), mode, Hq, Hkv, D)
    forms = {}
    for name, workgroups in made:
        m = re.search(r"attn_(fwd|bwd_dq)_head_kernelILi\d+ELb0ELi(\d)ELb([01])E", name)
        if m:
            forms[m[1]] = "draw" if m[3] == "1" else of_grid[workgroups]
            assert m[3] == "0" or workgroups == 1024 // int(m[2])
        elif "attn_fwd_group" in name:
            forms["fwd"] = "group"
            assert workgroups == (items + items // 128 * 8 + 7) // 8 * 8
        elif "attn_bwd_dkv_kernel" in name:
            column_workgroups = workgroups
        elif "attn_bwd_dkv_reduce" in name:  # one workgroup for every part that a column may be cut into beyond its first
            n = Hkv * (blocks + workgroups)
            forms["columns"] = {n: False, n + n // 8: True}[column_workgroups]
    assert (forms["fwd"], forms["bwd_dq"], forms["columns"]) == (forward, dq, columns)


@pytest.mark.parametrize("lens,Hq,Hkv,mode,two", small.PLANS)
def test_launches_of_a_plan(launches, lens, Hq, Hkv, mode, two):
    names = [name for name, _ in launches(lens, [3] * len(lens), mode, Hq, Hkv, 64, before=["plan"])]
    form = "ILb%dEE" % two
    assert [f for n in names if (f := re.search("plan_(?:lists|bwd_order)_kernel(I.*?EE)", n))] and all(form in n for n in names if "plan_" in n), names


@pytest.mark.parametrize("lens,Hq,Hkv,D,mode,one", small.AT_ONCE)
def test_launches_of_scores_with_a_selection(launches, lens, Hq, Hkv, D, mode, one):
    names = [name for name, _ in launches(lens, [3] * len(lens), mode, Hq, Hkv, D, before=["plan"])]
    forms = [f[0] for n in names if (f := re.search("score_select_kernel|score_kernel|topk_kernel", n))]
    assert forms == (["score_select_kernel"] if one else ["score_kernel", "topk_kernel"])
