"""Launch shapes of problems that are too large to run in a test: the library's calls in a process whose HIP launch calls only write
down what would be launched (CPU only; no buffer is read)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CALLS = """
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
import numpy as np
from paper_2604_13847_amd import binding as sb
S, L = 24, 65536
pb = sb.Problem(np.arange(S + 1) * L, [4] * S, 64, 64, 64, dtype=sb.SB_F32)
pb.c.cu_seqlens_dev = pb.c.topk_dev = 4096
b, lib, p = C.c_void_p(4096), sb.lib(), pb.ref()
sb._check(lib.sb_block_scores(p, b, b, None, b, b, None))
sb._check(lib.sb_select_topk(p, b, b, b, b, None))
sb._check(lib.sb_plan_worklist(p, b, b, b, None))
sb._check(lib.sb_sparse_attn_fwd(p, b, b, b, b, b, b, b, b, b, None))
sb._check(lib.sb_sparse_attn_bwd(p, b, b, b, b, b, b, b, b, b, b, b, b, b, None))
out = np.zeros((256, 6), dtype=np.uint32)
n = shim.recorded_launches(out.ctypes.data_as(C.c_void_p))
assert 0 < n <= 256, n
for l in out[:n].tolist():
    print("launch", *l)
"""


def test_launches_of_a_large_float32_problem_stay_within_the_limits(tmp_path):
    """1.6 million tokens on 64 heads in float32 (about 260 GB with gradients and workspaces): a HIP launch takes fewer than 2^32
    threads per dimension, and the tensors that are converted together have 4.8e9 (forward) and 6.4e9 (backward) quadruples."""
    shim = str(tmp_path / "record_launches.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(ROOT, "tests", "launch", "record_launches.c")], check=True)
    r = subprocess.run([sys.executable, "-c", CALLS, shim], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    launches = [tuple(map(int, l.split()[1:])) for l in r.stdout.splitlines() if l.startswith("launch ")]
    assert len(launches) >= 10
    for l in launches:
        assert all(1 <= g and g * t < 2 ** 32 for g, t in zip(l[:3], l[3:])) and l[1] <= 65535 and l[2] <= 65535, l


STEP = """
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
import numpy as np
from paper_2604_13847_amd import binding as sb
pb = sb.Problem([0, 64000], [2], 1, 1, 128)
pb.c.cu_seqlens_dev = pb.c.topk_dev = 4096
b, lib, p = C.c_void_p(4096), sb.lib(), pb.ref()
sb._check(lib.sb_plan_worklist(p, b, b, b, None))
sb._check(lib.sb_sparse_attn_bwd(p, b, b, b, b, b, b, b, b, b, b, b, b, b, None))
out = np.zeros((256, 6), dtype=np.uint32)
for l in out[:shim.recorded_launches(out.ctypes.data_as(C.c_void_p))].tolist():
    print("launch", *l)
"""


def test_columns_walked_by_several_workgroups_keep_the_launch_small(tmp_path):
    """1000 columns of two or three tiles, one of which could have 1000: room for its parts must not multiply the launch (an item's
    workgroups that find no part to walk, 68 for each here, keep the others off their XCDs)."""
    shim = str(tmp_path / "record_launches.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(ROOT, "tests", "launch", "record_launches.c")], check=True)
    r = subprocess.run([sys.executable, "-c", STEP, shim], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    launches = [tuple(map(int, l.split()[1:])) for l in r.stdout.splitlines() if l.startswith("launch ")]
    assert len(launches) >= 5 and max(x * y * z for x, y, z, *_ in launches) <= 8192, launches
