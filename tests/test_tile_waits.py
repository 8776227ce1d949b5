"""The tile kernels' LDS ring, read from the code the compiler makes of it: a
wait that ends a stage must leave outstanding no more memory operations than
that stage issued, so that the stage before has arrived whatever the order of
its loads.  (A load whose result is never used is deleted, and a wait counted
with it then reaches into the stage before.)  No GPU."""
import os
import re
import subprocess

import pytest

from paper_2605_30876_amd import build

LOAD = re.compile(r"(global|buffer|flat|scratch)_(load|store)")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "ffn.s")
    cmd = [build.hipcc(), "-x", "hip", "-S", "--cuda-device-only", os.path.join(build.CSRC, "ffn.hip"), "-o", out]
    subprocess.run(cmd + build._flags(False), check=True, capture_output=True, timeout=600)
    with open(out, encoding="utf-8") as f:
        return f.read()


def _stages(body):
    """(direct-to-LDS loads, memory operations, vmcnt at the barrier) of every barrier-to-barrier run of code."""
    out, lds, ops, wait = [], 0, 0, None
    for line in (l.strip() for l in body.splitlines()):
        if LOAD.match(line):
            ops += 1
            lds += "_load_lds" in line
            wait = None
        elif line.startswith("s_waitcnt"):
            m = re.search(r"vmcnt\((\d+)\)", line)
            if m:
                wait = int(m.group(1))
        elif line.startswith("s_barrier"):
            out.append((lds, ops, wait))
            lds, ops, wait = 0, 0, None
    return out


def test_stage_waits_cover_the_stage_before(assembly):
    kernels = re.findall(r"^(_Z\S*ffn_tile_bf16_kernel\S*):(.*?)\.size", assembly, re.S | re.M)
    assert len(kernels) == 5
    for name, body in kernels:
        stages = _stages(body)
        assert sum(lds > 0 for lds, _, _ in stages) >= 8 * 4, name  # eight bodies: prologue and three stages
        for i, (lds, ops, wait) in enumerate(stages):
            if wait is not None:
                assert ops >= wait, f"{name}: barrier {i} waits for vmcnt({wait}) after {ops} operations ({lds} to LDS)"
