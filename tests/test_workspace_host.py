"""The library's host side on a device that is not there (fake_hip.cpp): what it allocates for which call, what it does when memory
is short, and which launches it makes.  Every test runs in a process of its own, in which the HIP runtime's names resolve to
the fake."""
import functools
import json
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, json, sys
sys.path.insert(0, {root!r})
from paper_2605_16360_amd import binding as pk  # torch, which comes with it, keeps the runtime it has found
fake = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_budget.argtypes = [ctypes.c_size_t]
fake.fake_used.restype = fake.fake_peak.restype = ctypes.c_size_t
fake.fake_launches.restype = ctypes.c_char_p
lib = pk.load()
P = ctypes.c_void_p(1 << 41)  # any address: nothing reads it
LLAMA, QWEN, QWEN32B = (16, 32, 8, 64, 32, 8, 128), (24, 14, 2, 64, 28, 4, 128), (28, 12, 2, 128, 64, 8, 128)

kept = []

def context(shape, weights=False, reduce=0):
    cfg = pk.make_config(*shape)
    cfg.reduce = reduce
    ctx = pk.proxykv_create(cfg)
    if weights:
        n = pk.proxykv_mapper_weight_count(cfg)
        blob = (ctypes.c_float * n)(*([1.0] * n)) if n < 1000 else (ctypes.c_float * n)()
        assert lib.proxykv_set_mapper_weights(ctx.handle, blob, n) == 0
    kept.append(ctx)  # destroyed with its last reference
    return ctx.handle

def launches(part=""):
    out = [l for l in fake.fake_launches().decode().splitlines() if part in l]
    return [(l.split()[0], *map(int, l.split()[-4:])) for l in out]
"""


@functools.lru_cache(maxsize=None)
def fake_so():
    import tempfile
    so = os.path.join(tempfile.mkdtemp(), "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so], check=True)
    return so


def run(code):
    """Runs `code`, which leaves its answer in `out`, and returns that."""
    script = PRELUDE.format(so=fake_so(), root=ROOT) + textwrap.dedent(code) + "\nprint('OUT' + json.dumps(out))\n"
    r = subprocess.run([sys.executable, "-c", script], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads([l for l in r.stdout.splitlines() if l.startswith("OUT")][-1][3:])


def test_the_max_form_allocates_row_sums_and_nothing_else():
    """Only the sum and the causal form have column sums of several workgroups to keep."""
    out = run("""
        out = {}
        for n in (512, 8192):
            for what in ("max", "sum", "self"):
                used = fake.fake_used()
                h = context(LLAMA, reduce=1 if what == "sum" else 0)
                rc = lib.proxykv_score_self(h, P, P, 0, n, P, None) if what == "self" else lib.proxykv_score(h, P, P, P, 0, n, n, 2048, P, None)
                assert rc == 0
                out[f"{what} {n}"] = fake.fake_used() - used
    """)
    for n in (512, 8192):
        rows = 16 * 32 * n
        lse = max(4 * rows, 8 * min(8 * rows, 768 * 256))  # a float per query, or a pair per query and sharing workgroup
        assert out[f"max {n}"] == lse
        assert out[f"sum {n}"] == out[f"self {n}"] > lse
