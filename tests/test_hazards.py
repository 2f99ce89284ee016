"""The attention kernels issue buffer loads from inline assembly, where the compiler does not look for hazards: a scalar register written by a
vector instruction (v_readlane, v_readfirstlane) must not be read by a vector-memory instruction within five wait states.  The
assembly that the compiler makes of the present sources is scanned for it."""
import os
import re
import subprocess

import pytest

from paper_2604_13847_amd import build

WAIT_STATES = 5
LOAD = re.compile(r"buffer_load_dword\S* v\d+, s\[(\d+):(\d+)\], 0 offen")
WRITE = re.compile(r"v_read(?:lane|firstlane)_b32 s(\d+),")


def hazards(lines):
    seen, loads, bad = [], 0, []
    for line in (l.strip() for l in lines):
        if not line or line[0] in ";.":
            continue
        m = LOAD.match(line)
        if m:
            loads += 1
            states = 0
            for before in reversed(seen[-WAIT_STATES:]):
                w = WRITE.match(before)
                if w and int(m[1]) <= int(w[1]) <= int(m[2]) and states < WAIT_STATES:
                    bad.append((before, line, states))
                nop = re.match(r"s_nop (\d+)", before)
                states += int(nop[1]) + 1 if nop else 1
        seen.append(line)
    return loads, bad


def test_the_scan_sees_a_hazard():
    load = "buffer_load_dwordx4 v1, s[20:23], 0 offen offset:0 lds"
    assert hazards(["v_readlane_b32 s22, v1, 3", "s_nop 2", load])[1]
    assert not hazards(["v_readlane_b32 s22, v1, 3", "s_nop 4", load])[1]
    assert not hazards(["v_readlane_b32 s24, v1, 3", load])[1]


@pytest.mark.parametrize("source", ["sb_attn_fwd.hip", "sb_attn_bwd.hip"])
def test_no_vector_write_right_before_a_load_that_reads_it(source, tmp_path):
    out = str(tmp_path / "a.s")
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
    loads, bad = hazards(open(out).read().splitlines())
    assert loads > 100 and not bad, bad[:3]
