"""The split Top-K's workgroups meet in a per-row histogram: each adds its bins, then takes a ticket, and the last to arrive
reads the histogram.  Nothing but a wait for outstanding memory operations orders a wave's adds before the ticket, and a
run cannot show that it is missing (the adds are nearly always done by then), so the compiled code is checked: in every
pass kernel `s_waitcnt vmcnt(0)` stands between the last add without a result and the barrier in front of the ticket."""
import os
import re
import subprocess

import pytest

from paper_2605_16360_amd import build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "topk.s")
    r = subprocess.run([build._hipcc(), *build.FLAGS, "-x", "hip", "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, "topk.hip"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read()


def test_every_pass_waits_for_its_adds_before_the_ticket(assembly):
    kernels = re.findall(r"^(_ZN\w*mw_pass_kernel\w*):(.*?)^\.Lfunc_end", assembly, re.M | re.S)
    assert len(kernels) == 7  # three passes of 11 bits, four of 8
    for name, body in kernels:
        ops = re.findall(r"^\s+(global_atomic_add\b.*|s_barrier\b|s_waitcnt\b.*)$", body, re.M)
        adds = [i for i, op in enumerate(ops) if op.startswith("global_atomic_add")]
        bins = [i for i in adds if "sc0" not in ops[i]]  # sc0: the old value is returned
        ticket = next(i for i in adds if i > bins[-1])
        barriers = [i for i in range(bins[-1], ticket) if ops[i].startswith("s_barrier")]
        assert barriers, name
        assert any("vmcnt(0)" in op for op in ops[bins[-1]:barriers[-1]]), name
