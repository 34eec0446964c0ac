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


def test_mapper_memory_is_bounded():
    """Batches of layers hold about 6 KB per window row and no more rows than all layers have, or 2 x 65 536, or, where layers are
    longer than half of that, four of them: below 1 GB up to 16 384 tokens, and from there on less than four layers at the 12 KB
    per row that one layer at a time on four streams took.  proxykv_workspace_bytes counts what proxykv_reserve allocates."""
    out = run("""
        out = []
        for shape in (LLAMA, QWEN, QWEN32B):
            for n in (512, 1500, 2500, 4096, 8192, 16384, 32768, 65536, 170000):
                used = fake.fake_used()
                h = context(shape, weights=True)
                weights = fake.fake_used()
                assert lib.proxykv_map(h, P, n, P, None) == 0
                size = ctypes.c_size_t()
                assert lib.proxykv_workspace_bytes(ctypes.byref(pk.make_config(*shape)), n, n, ctypes.byref(size)) == 0
                total = ctypes.c_size_t(fake.fake_used() - weights)
                before = fake.fake_used()
                assert lib.proxykv_reserve(h, n, n) == 0
                out.append((shape[0], n, total.value, size.value, total.value + fake.fake_used() - before))
    """)
    for layers, n, mapper, said, reserved in out:
        windows = 1 if n <= 2048 else -(-(n - 2048) // 1024) + 1
        rows = -(-(n + (windows - 1) * 1024) // 256) * 256
        assert mapper <= max(min(layers * rows, 2 * 65536), (4 if rows <= 65536 else 2) * rows) * 7.5 * 1024 + 20e6, (layers, n, mapper)
        assert n > 16384 or mapper < 1e9, (layers, n, mapper)
        assert n < 16384 or mapper < 4 * rows * 12 * 1024, (layers, n, mapper)
        assert said == reserved, (layers, n, said, reserved)


def test_large_tiles_have_no_room_for_the_rows_they_keep_to_themselves():
    """x, its fp16 copy, q with k and v are 6 KB per row, whatever d_ffn; the FFN's hidden rows and the second fp16 row belong to short
    batches only, for which a longer call's workspace still has room in one piece."""
    out = run("""
        out = []
        for d_ffn in (2048, 8192):
            for n in (4096, 8192, 32768):
                cfg = pk.make_config(*LLAMA)
                cfg.d_ffn = d_ffn
                ctx = pk.proxykv_create(cfg)
                kept.append(ctx)
                count = pk.proxykv_mapper_weight_count(cfg)
                assert lib.proxykv_set_mapper_weights(ctx.handle, (ctypes.c_float * count)(), count) == 0
                before = fake.fake_used()
                assert lib.proxykv_map(ctx.handle, P, n, P, None) == 0
                used = fake.fake_used() - before
                batches = []
                for short in (80, 150, 160):
                    launches()
                    assert lib.proxykv_map(ctx.handle, P, short, P, None) == 0
                    batches.append([l[2] for l in launches("stage3_kernel")])
                assert fake.fake_used() - before == used
                out.append((d_ffn, n, used, batches))
    """)
    for d_ffn, n, used, batches in out:
        rows = {4096: 16 * 6144, 8192: 2 * 4 * 14336, 32768: 2 * 2 * 63488}[n]  # in flight on both lanes
        short = 16 * 256 * 2 * max(2048, d_ffn) + 16 * 256 * 2048
        assert used <= rows * 6.3 * 1024 + short, (d_ffn, n, used)
        assert batches == [[16]] * 3, (d_ffn, n, batches)


def test_mapper_makes_do_with_less_memory():
    """A device with room for one layer's activations runs all layers one at a time; with less the call is refused; and a workspace
    that the mapper has taken is given up when another buffer does not fit beside it."""
    out = run("""
        out = {}
        n = 8192
        one = ctypes.c_size_t()
        h = context((1,) + LLAMA[1:4] + (1,) + LLAMA[5:], weights=True)
        base = fake.fake_used()
        assert lib.proxykv_map(h, P, n, P, None) == 0
        layer = fake.fake_used() - base
        for room in (0.9, 1.1, 2.3, 5.0):
            h = context(LLAMA, weights=True)
            fake.fake_budget(fake.fake_used() + int(room * layer))
            launches()
            for again in range(2):
                rc = lib.proxykv_map(h, P, n, P, None)
                out[f"{room} {again}"] = [rc, [l[2] for l in launches("stage3_kernel")]]
            fake.fake_budget((1 << 63) - 1)
        # score in fp32 after the mapper: its bf16 copies fit only if the mapper gives way.  They and the row sums are 822 MB, what the
        # mapper holds 732 MB, so that beside two layers' room (186 MB) one layer's is left for the mapper's next call.
        h = context(LLAMA, weights=True)
        assert lib.proxykv_map(h, P, n, P, None) == 0
        fake.fake_budget(fake.fake_used() + 2 * layer)
        out["score"] = lib.proxykv_score(h, P, P, P, 1, n, n, 2048, P, None)
        launches()
        out["map"] = lib.proxykv_map(h, P, n, P, None)
        out["layers"] = [l[2] for l in launches("stage3_kernel")]
    """)
    assert out["0.9 0"][0] == out["0.9 1"][0] == -3  # PROXYKV_ENOMEM
    for room, most in (("1.1", 1), ("2.3", 1), ("5.0", 2)):
        for again in "01":
            rc, layers = out[f"{room} {again}"]
            assert rc == 0 and sum(layers) == 16 and max(layers) == most, (room, again, layers)
    assert out["score"] == out["map"] == 0 and sum(out["layers"]) == 16


def test_no_call_allocates_after_a_longer_one():
    """A context that has served a call (or proxykv_reserve) serves every shorter one from the same memory, so that it can be captured:
    whatever the plan of the shorter one would rather have, all layers are covered and nothing is allocated."""
    out = run("""
        out = []
        lengths = [5, 200, 700, 1024, 1500, 2048, 2049, 3000, 4097, 4608, 5000, 8192, 11500, 16384, 30000]
        for shape in (LLAMA, QWEN, QWEN32B, (33, 4, 2, 64, 33, 4, 128), (3, 4, 2, 64, 3, 4, 128)):
            for longest in lengths[5::3]:
                for reserved in (False, True):
                    h = context(shape, weights=True)
                    if reserved:
                        assert lib.proxykv_reserve(h, longest, longest) == 0
                    calls = 0
                    for n in [longest] + [n for n in lengths if n < longest]:
                        launches()
                        before = fake.fake_mallocs()
                        rc = [lib.proxykv_map(h, P, n, P, None), lib.proxykv_score(h, P, P, P, 0, n, n, 512, P, None),
                              lib.proxykv_score_self(h, P, P, 0, n, P, None)]
                        layers = sum(l[2] for l in launches("stage3_kernel"))
                        if n < longest or reserved:
                            out.append((rc, layers == shape[0], fake.fake_mallocs() - before, shape, longest, n))
    """)
    assert len(out) > 200
    for rc, covered, mallocs, shape, longest, n in out:
        assert rc == [0, 0, 0] and covered and mallocs == 0, (shape, longest, n, mallocs)


def test_short_maps_after_a_long_one_keep_their_batches():
    """A longer call holds few layers of many rows at a time, which is room for many layers of few rows: a shorter call makes the batches
    that it would make in a context of its own."""
    out = run("""
        out = []
        for shape in (LLAMA, QWEN, QWEN32B):
            def batches(h, n):
                launches()
                assert lib.proxykv_map(h, P, n, P, None) == 0
                return [l[2] for l in launches("stage3_kernel")]
            fresh = {n: batches(context(shape, weights=True), n) for n in (80, 160, 1000, 1500, 2000)}
            for longest in (8192, 32768, 170000):
                h = context(shape, weights=True)
                batches(h, longest)
                out += [(shape[0], longest, n, batches(h, n), fresh[n]) for n in fresh]
    """)
    assert len(out) == 45
    for layers, longest, n, got, own in out:
        assert got == own, (layers, longest, n, got, own)


def test_mapper_deals_few_layers_to_both_lanes():
    """More rows than fill the chip in one turn go to two streams also where one batch could hold all layers: three layers of 3000
    tokens one behind the other took longer than side by side.  Short ones stay in one batch."""
    out = run("""
        out = {}
        for layers, n in ((3, 3000), (4, 4500), (16, 1500), (5, 9000), (2, 1500), (16, 250), (1, 30000)):
            h = context((layers, 4, 2, 64, layers, 4, 128), weights=True)
            assert lib.proxykv_map(h, P, n, P, None) == 0
            out[f"{layers} {n}"] = [l[2] for l in launches("stage3_kernel")]
    """)
    assert out == {"3 3000": [1, 2], "4 4500": [2, 2], "16 1500": [8, 8], "5 9000": [2, 3], "2 1500": [2], "16 250": [16],
                   "1 30000": [1]}


def test_topk_and_column_sums_make_do_with_less_memory():
    """The wide histograms of long rows take five times the memory of the narrow ones, the column sums of several workgroups per key block
    take some where there were none: both are done without where they do not fit, on the next call too, and no call of
    fewer or shorter rows than one before it allocates."""
    out = run("""
        out = {}
        h = context(LLAMA)
        rows, n = 1000, 170000
        fake.fake_budget(fake.fake_used() + 10 * 1000 * 1000)  # narrow 8.3 MB, wide 41 MB
        out["topk"] = [[lib.proxykv_topk(h, P, rows, n, 1000, P, None), sorted({l[0] for l in launches("mw_pass_kernel")})] for _ in range(2)]
        h = context(QWEN, reduce=1)
        fake.fake_budget(fake.fake_used() + 20 * 1000 * 1000)  # row sums 8 MB, column sums 19 MB
        out["sum"] = []
        for _ in range(2):
            launches()
            before = fake.fake_mallocs()
            rc = lib.proxykv_score(h, P, P, P, 0, 6001, 6001, 2048, P, None)
            out["sum"].append([rc, len(launches("sum_parts_kernel")), fake.fake_mallocs() - before])
        fake.fake_budget((1 << 63) - 1)
        h = context(QWEN, reduce=1)
        assert lib.proxykv_score(h, P, P, P, 0, 6001, 6001, 2048, P, None) == 0
        out["parts"] = len(launches("sum_parts_kernel"))
        out["mallocs"] = []
        for big, small in (((257, 45000), (256, 45000)), ((600, 60000), (100, 50000)), ((5, 300000), (1, 299999)), ((112, 170000), (40, 80000))):
            h = context(LLAMA)
            assert lib.proxykv_topk(h, P, big[0], big[1], 9, P, None) == 0
            before = fake.fake_mallocs()
            assert lib.proxykv_topk(h, P, small[0], small[1], 9, P, None) == 0
            assert lib.proxykv_topk_pooled(h, P, small[0], 1, small[1], 9, P, P, None) == 0
            out["mallocs"].append(fake.fake_mallocs() - before)
    """)
    for rc, kernels in out["topk"]:
        assert rc == 0 and len(kernels) == 4 and all("ILi8E" in k for k in kernels)
    assert out["sum"][0][:2] == [0, 0] and out["sum"][1] == [0, 0, 0]
    assert out["parts"] == 1 and out["mallocs"] == [0, 0, 0, 0]


def test_launches_of_many_rows_stay_within_the_runtime():
    """A launch counts its threads per dimension in 32 bits: more rows than 1024 threads each allow are marked with fewer, and more
    (layer, head) pairs than a wave each allows are counted by waves that take several."""
    out = run("""
        out = {}
        h = context(LLAMA)
        out["mask"] = [lib.proxykv_mask(h, P, 5 * 1000 * 1000, 8192, 1, P, None), launches("mask_kernel")]
        out["pooled"] = [lib.proxykv_topk_pooled(h, P, 2000, 36000, 1, 1, P, P, None), launches("head_counts_kernel")]
        out["few"] = [lib.proxykv_topk_pooled(h, P, 3, 5, 100, 10, P, P, None), launches("head_counts_kernel")[0][1]]
    """)
    assert out["mask"][0] == 0 and out["mask"][1][0][1:] == [5000000, 1, 1, 256]
    assert out["pooled"][0] == 0 and out["pooled"][1][0][1] * 64 <= 0xffffffff
    assert out["few"] == [0, 15]


def test_topk_masks_give_way_before_the_histograms_do():
    """1000 rows of 170 000 scores: 106 MB of scratch memory with two bits per score, 41 MB without them, 8 MB with the narrow histograms.
    Where the bits do not fit the wide histograms stay, and the mapper keeps its workspace, as long as they fit beside it."""
    out = run("""
        out = {}
        rows, n = 1000, 170000
        for room in (9, 50, 120):
            h = context(LLAMA)
            fake.fake_budget(fake.fake_used() + room * 1000 * 1000)
            before = fake.fake_used()
            out[str(room)] = [[lib.proxykv_topk(h, P, rows, n, 1000, P, None), len(launches("mw_pass_kernelILi11E"))] for _ in range(2)]
            out[f"{room} MB"] = (fake.fake_used() - before) // 1000000
            fake.fake_budget((1 << 63) - 1)
        h = context(LLAMA, weights=True)
        assert lib.proxykv_map(h, P, 4096, P, None) == 0
        fake.fake_budget(fake.fake_used() + 50 * 1000 * 1000)
        before = fake.fake_used()
        out["beside"] = [lib.proxykv_topk(h, P, rows, n, 1000, P, None), len(launches("mw_pass_kernelILi11E")), (fake.fake_used() - before) // 1000000]
        mallocs = fake.fake_mallocs()
        assert lib.proxykv_map(h, P, 4096, P, None) == 0
        out["map again"] = fake.fake_mallocs() - mallocs
    """)
    assert out == {"9": [[0, 0]] * 2, "9 MB": 8, "50": [[0, 3]] * 2, "50 MB": 41, "120": [[0, 3]] * 2, "120 MB": 106,
                   "beside": [0, 3, 41], "map again": 0}


def test_short_launches_of_pass_1_take_the_wide_tiles():
    """28 x 12 heads of 128: pass 1's 16-column tiles gain in long launches only (300 keys 54.8 us with 32 columns, 57.1 with 16)."""
    out = run("""
        ctx = context(QWEN32B)
        out = {}
        for n, n_q in ((300, 300), (768, 768), (1500, 300), (900, 900), (4000, 500), (10007, 10007)):
            launches()
            assert lib.proxykv_score(ctx, P, P, P, 0, n, n_q, 4096, P, None) == 0
            out[f"{n} {n_q}"] = [l[0] for l in launches("score_lse_kernel")]
    """)
    for case, wide in (("300 300", True), ("768 768", True), ("1500 300", True), ("900 900", False), ("4000 500", False), ("10007 10007", False)):
        assert len(out[case]) == 1 and ("ILi128ELi2ELi32E" in out[case][0]) == wide, (case, out[case])


def test_in_place_compaction_of_short_rows_has_more_workgroups():
    """Tokens of 256 bytes move in one piece (two workgroups a row: K and V) where rows are many and long, in two where they are few or short
    (256 rows, 150 kept of 1500: 18.3 us in two, 19.3 in one); with shared budgets in one whatever the length."""
    out = run("""
        out = {}
        h = context(LLAMA)
        for rows, k in ((256, 512), (256, 513), (255, 600)):
            launches()
            assert lib.proxykv_compact_inplace(h, P, P, P, rows, 2000, k, 128, None) == 0
            out[f"{rows} {k}"] = [l[1:3] for l in launches("compact_inplace_kernel")]
        for layers, heads, k in ((64, 4, 100), (51, 5, 100)):
            launches()
            assert lib.proxykv_compact_pooled(h, P, P, P, P, layers, heads, 2000, k, 128, None) == 0
            out[f"{layers} {heads}"] = [l[1:3] for l in launches("compact_inplace_kernel")]
    """)
    assert out == {"256 512": [[256, 4]], "256 513": [[256, 2]], "255 600": [[255, 4]], "64 4": [[256, 2]], "51 5": [[255, 4]]}


def test_a_captured_in_place_compaction_holds_nothing_of_the_context():
    """A graph may outlive what the context's calls behind it grow, and the context itself: a captured call moves whole rows with the caller's
    pointers alone, also where the context has room for the counters of an eager one, which uses them."""
    out = run("""
        out = []
        h = context(LLAMA)
        for reserved in (False, True):
            if reserved:
                assert lib.proxykv_reserve(h, 8192, 8192) == 0
            for pooled in (False, True):
                for capturing in (0, 1, 0):
                    fake.fake_capturing(capturing)
                    launches()
                    before = fake.fake_mallocs()
                    rc = (lib.proxykv_compact_pooled(h, P, P, P, P, 32, 8, 8192, 4096, 128, None) if pooled else
                          lib.proxykv_compact_inplace(h, P, P, P, 256, 8192, 4096, 128, None))
                    names = "".join(sorted(l[0] for l in launches()))
                    out.append((rc, capturing, "compact_parts_kernel" in names, "compact_inplace_kernel" in names, capturing and fake.fake_mallocs() - before))
    """)
    assert len(out) == 12
    for rc, capturing, parts, whole, mallocs in out:
        assert (rc, parts, whole, mallocs) == (0, not capturing, bool(capturing), 0), out


def test_in_place_counters_take_nothing_from_the_topk():
    """Where there is no memory for the in-place compaction's counters (15 MB of them here) the call moves whole rows, and the Top-K's workspace stays: rows
    that fitted before are selected without an allocation, on the narrow histograms too."""
    out = run("""
        out = []
        for narrow in (False, True):
            for pooled in (False, True):
                h = context(LLAMA)
                fake.fake_budget(fake.fake_used() + (1000 * 1000 if narrow else 1 << 40))
                assert lib.proxykv_topk(h, P, 40, 60000, 9, P, None) == 0
                fake.fake_budget(fake.fake_used() + 1000)
                launches()
                rc = (lib.proxykv_compact_pooled(h, P, P, P, P, 8000, 5, 40000, 30000, 128, None) if pooled else
                      lib.proxykv_compact_inplace(h, P, P, P, 40000, 40000, 30000, 128, None))
                whole = len(launches("compact_inplace_kernel"))
                before = fake.fake_mallocs()
                again = lib.proxykv_topk(h, P, 40, 60000, 9, P, None)
                out.append((rc, whole, again, fake.fake_mallocs() - before))
                fake.fake_budget((1 << 63) - 1)
    """)
    assert out == [[0, 1, 0, 0]] * 4


def test_in_place_calls_of_several_streams_count_apart():
    """In-place calls of one context on several streams, on caches of their own, need not follow each other, so each stream has counters of its own, the same
    again on its next call and apart from the others' also after one of them had to have more.  The streams beyond
    those that have some, and the per-thread default stream, whose handle is the same in every thread, move whole rows."""
    out = run("""
        out = {}
        fake.fake_argument.restype = ctypes.c_uint64
        fake.fake_watch(b"compact_parts_kernel", 9)
        h = context(LLAMA)
        def counters(stream, rows=256, K=4096):
            launches()
            assert lib.proxykv_compact_inplace(h, P, P, P, rows, 8192, K, 128, ctypes.c_void_p(stream)) == 0
            parts = launches("compact_parts_kernel")
            return fake.fake_argument() if parts else 0
        out["first"] = [counters(1000 + i) for i in range(40)]
        out["again"] = [counters(1000 + i) for i in range(40)]
        size = 4 * 2 * 256 * 8  # seven parts and the counter for every row, K and V
        out["apart"] = all(abs(a - b) >= size for a in out["first"] for b in out["first"] if a and b and a != b)
        mallocs = fake.fake_mallocs()
        out["more"] = [counters(1000 + i, rows=600) for i in (0, 1, 0)]
        out["grown"] = fake.fake_mallocs() - mallocs
        out["older"] = [counters(1000 + i) for i in range(3)]
        out["per thread"] = counters(2)
        h = context(LLAMA)
        out["default"] = [counters(0), counters(2), counters(0)]
    """)
    with_some = [c for c in out["first"] if c]
    assert len(with_some) == len(set(with_some)) == 32 and out["first"] == with_some + [0] * 8
    assert out["again"] == out["first"] and out["apart"] and out["grown"] == 1
    a, b, c = out["more"]
    assert a == c and abs(a - b) >= 4 * 2 * 600 * 8 and len(set(out["older"])) == 3
    assert out["per thread"] == 0
    assert out["default"][0] == out["default"][2] != 0 and out["default"][1] == 0


def test_in_place_calls_of_several_threads():
    """Four threads and a context: none loses its counters while another makes room for its own.  (A block has less than twice what is asked for, the
    ones before it together less than it.)"""
    out = run("""
        import threading
        out = []
        h = context(LLAMA)
        def work(stream):
            for k in range(1000, 8000, 50):
                out.append(lib.proxykv_compact_inplace(h, P, P, P, 256, 8192, k, 128, ctypes.c_void_p(stream)))
        before = fake.fake_used()
        threads = [threading.Thread(target=work, args=(1000 + i,)) for i in range(4)]
        for t in threads: t.start()
        for t in threads: t.join()
        grew = fake.fake_used() - before
        kept.clear()
        out = [sorted(set(out)), len(out), grew < 4 * 32 * 4 * 2 * 256 * 14, fake.fake_used() <= before]
    """)
    assert out == [[0], 560, True, True]


def test_in_place_compaction_in_parts_only_where_whole_rows_are_slower():
    """Few short rows are moved before a second launch has begun (D = 256, one row that keeps 1440 tokens: 10.5 us whole, 12.8 in parts), and 280 parts are two
    turns on 256 places; the tests of parts on a GPU keep enough for them."""
    out = run("""
        out = []
        h = context(LLAMA)
        def parts(layers, heads, D, K, pooled, N=None):
            launches()
            N = N or K + 5
            rc = (lib.proxykv_compact_pooled(h, P, P, P, P, layers, heads, N, K, D, None) if pooled else
                  lib.proxykv_compact_inplace(h, P, P, P, layers * heads, N, K, D, None))
            assert rc == 0
            return len(launches("compact_parts_kernel"))
        out.append([parts(*c) for c in ((1, 1, 256, 1440, 0), (1, 4, 256, 1440, 0), (4, 7, 256, 1440, 0), (1, 4, 128, 1024, 1), (4, 7, 256, 512, 1),
                                        (1, 4, 256, 1024, 1))])
        out.append([parts(*c) for c in ((1, 1, 256, 1984, 0), (1, 4, 256, 1984, 0), (1, 1, 128, 2048, 0), (1, 4, 128, 1500, 1), (4, 7, 64, 2048, 1), (28, 4, 128, 1920, 0),
                                        (28, 4, 128, 1500, 1), (32, 8, 128, 1024, 0), (64, 8, 128, 6172, 0), (64, 8, 128, 6172, 1), (32, 8, 8, 20000, 0))])
        # as in test_gpu_parity.py
        out.append([parts(*c) for c in ((1, 3, 128, 1921, 0), (1, 256, 128, 960, 0), (1, 256, 128, 1500, 0), (1, 2, 256, 2000, 0), (1, 2, 72, 3411, 0), (1, 1, 8, 30720, 0), (1, 256, 64, 1920, 0),
                                        (1, 2, 256, 1919, 0), (1, 2, 256, 1920, 0), (1, 2, 256, 1921, 0), (1, 2, 256, 2241, 0), (1, 130, 128, 3000, 1, 4000),
                                        (2, 70, 64, 4000, 1, 5000), (3, 2, 128, 1500, 1, 4000), (1, 4, 128, 3000, 0), (1, 3, 128, 4000, 0), (1, 40, 128, 3000, 0), (1, 64, 128, 2500, 0))])
        # what is reserved is enough for every number of kept tokens
        h = context(LLAMA)
        assert lib.proxykv_reserve(h, 9000, 64) == 0
        before = fake.fake_mallocs()
        for K in range(1, 9001, 7):
            parts(32, 8, 128, K, K % 2, 9000)
        out.append(fake.fake_mallocs() - before)
    """)
    assert out[0] == [0] * 6 and out[1] == [1] * 11 and out[2] == [1] * 18 and out[3] == 0


def test_fp32_scores_are_rounded_in_front_where_several_xcds_read_a_share_of_the_keys():
    """Pass 1 rounds fp32 keys itself only where that does not read much of them in twice the bytes: a share of a KV head's keys goes to one XCD (shares make
    eight workgroups per query block), or each XCD that reads it does so for several workgroups, or the keys are few."""
    out = run("""
        out = []
        for L, H_q, H_kv, N, N_q, self in ((11, 32, 8, 2000, 256, 0), (11, 32, 8, 4096, 128, 0), (9, 32, 8, 4096, 64, 0), (9, 32, 8, 400, 256, 0), (8, 32, 8, 2000, 64, 0),
                                           (20, 8, 4, 4096, 64, 0), (28, 12, 2, 4096, 64, 0), (4, 32, 8, 4096, 512, 0), (14, 14, 2, 4096, 64, 0), (11, 32, 8, 256, 256, 0),
                                           (11, 32, 8, 300, 300, 1), (1, 4, 2, 8000, 128, 0), (16, 32, 8, 512, 512, 0),
                                           (1, 4, 2, 512, 128, 0), (1, 4, 2, 4096, 4096, 0), (2, 32, 8, 4096, 256, 0), (3, 32, 8, 1600, 64, 0), (12, 16, 2, 4096, 64, 0),
                                           (16, 16, 16, 4096, 64, 0), (24, 14, 2, 1600, 256, 0), (9, 32, 8, 100, 256, 0), (9, 32, 8, 200, 64, 0), (8, 32, 8, 256, 64, 0),
                                           (1, 4, 2, 4000, 4000, 1), (4, 32, 8, 512, 256, 0), (8, 32, 8, 1000, 64, 0)):
            h = context((L, H_q, H_kv, 64, 1, 4, 128))
            launches()
            rc = lib.proxykv_score_self(h, P, P, 1, N, P, None) if self else lib.proxykv_score(h, P, P, P, 1, N, N_q, 2048, P, None)
            assert rc == 0
            out.append(len(launches("f32_to_bf16_kernel")))
    """)
    assert out == [1] * 13 + [0] * 13
