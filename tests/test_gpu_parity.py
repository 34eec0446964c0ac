"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded
inputs.  Integer and byte results are bit-exact; floating-point results are within
|gpu - ref| <= 2e-3 + 1e-2 * |ref| (bf16 inputs, fp32 accumulation)."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2605_16360_amd import binding as pk
from paper_2605_16360_amd import synth

pytestmark = pytest.mark.gpu
ATOL, RTOL = 2e-3, 1e-2


def assert_close(gpu: torch.Tensor, ref: torch.Tensor, what: str):
    g, r = gpu.detach().double().cpu(), ref.double()
    assert g.shape == r.shape, (g.shape, r.shape)
    assert bool(torch.isfinite(g).all()), f"{what}: non-finite values"
    err = (g - r).abs()
    bound = ATOL + RTOL * r.abs()
    worst = int(torch.argmax(err - bound))
    assert bool((err <= bound).all()), (f"{what}: max abs err {float(err.max()):.3e}, worst at flat {worst}: "
                                        f"gpu {float(g.flatten()[worst])} ref {float(r.flatten()[worst])}")


def _ctx(case, weights=None):
    ctx = pk.proxykv_create(pk.config_for_case(case))
    if weights is not None:
        pk.proxykv_set_mapper_weights(ctx, weights)
    return ctx


# ----------------------------------------------------------------------------------------------
# top-k and compaction: bit-exact
# ----------------------------------------------------------------------------------------------

@pytest.mark.parametrize("N,K", [(1, 1), (17, 5), (1000, 300), (1024, 1024), (1025, 1), (5000, 1500), (32771, 9830),
                                 (70001, 21000)])
def test_topk_bit_exact(N, K):
    ctx = _ctx(synth.CASES["tiny"])
    g = torch.Generator().manual_seed(N + K)
    s = torch.randn(7, N, generator=g)
    s[1] = torch.round(s[1] * 4) / 4             # heavy ties
    s[2] = 0.5                                   # all equal
    s[3] = torch.round(s[3])
    if N > 8:
        s[4, ::5] = float("nan")
        s[5, 1], s[5, 2], s[5, 3], s[5, 4] = -0.0, 0.0, float("inf"), float("-inf")
        s[5, 5:] = torch.where(s[5, 5:].abs() < 0.5, torch.zeros(()), s[5, 5:])
        s[5, 7::2] *= -1.0                       # produces -0.0 next to +0.0
    s[6] = s[6] * 1e-3 + 0.25                    # narrow range: many shared high radix digits
    ref = oracle.topk(s, K)
    got = pk.proxykv_topk(ctx, s.cuda(), K)
    torch.cuda.synchronize()
    assert torch.equal(got.cpu(), ref)


@pytest.mark.parametrize("N", [36863, 36864, 36865, 40000, 45057, 90113, 170000])
def test_topk_bit_exact_around_the_kernel_switch(N):
    """Rows of up to 36 864 scores are selected by one workgroup, longer ones are split into parts of at most 45 056
    (one part, two parts, three parts with a ragged last one, four parts)."""
    ctx = _ctx(synth.CASES["tiny"])
    g = torch.Generator().manual_seed(N)
    s = torch.randn(5, N, generator=g)
    s[1] = torch.round(s[1] * 3) / 3
    s[2] = -7.5
    s[3, N // 2:] = s[3, :N - N // 2].clone()        # every value twice: the tie rule decides half of the cut
    for K in (1, N // 3, N - 1, N):
        got = pk.proxykv_topk(ctx, s.cuda(), K)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), oracle.topk(s, K)), (N, K)


@pytest.mark.parametrize("rows,N", [(3, 255), (3, 2305), (3, 36861), (3, 36865), (600, 36868), (3, 45057), (2, 524293)])
def test_topk_ties_nan_thresholds_and_odd_lengths(rows, N):
    """Rows of a few distinct values (ties across the stretches of waves and parts), rows that are mostly NaN (the K-th
    largest is NaN), rows with both zeros and infinities, a constant row; lengths that leave a row off a 16-byte boundary,
    at the edge of the one-workgroup kernel, and few enough rows that one is cut into many parts.  proxykv_topk_static's
    histograms are narrower than proxykv_topk's for the long rows."""
    g = torch.Generator().manual_seed(N)
    distinct = 3 if rows > 2 else rows
    base = torch.randn(distinct, N, generator=g)
    base[0] = torch.randint(-2, 3, (N,), generator=g).float() * 0.0 + torch.randint(0, 4, (N,), generator=g).float()
    base[0, ::7] = -0.0
    base[1, torch.rand(N, generator=g) < 0.7] = float("nan")
    base[1, ::11] = float("inf")
    base[1, 1::13] = float("-inf")
    if distinct > 2:
        base[2] = 0.25
    s = base.repeat((rows + distinct - 1) // distinct, 1)[:rows].contiguous()
    ctx = _ctx(synth.CASES["tiny"])
    d = s.cuda()
    for K in sorted({1, max(1, N // 5), max(1, N // 2), N - 1 if N > 1 else 1, N}):
        ref = oracle.topk(base, K).repeat((rows + distinct - 1) // distinct, 1)[:rows]
        idx = pk.proxykv_topk(ctx, d, K)
        out = torch.empty_like(idx)
        pk.proxykv_topk_static(ctx, d, K, out)
        torch.cuda.synchronize()
        assert torch.equal(idx.cpu().long(), ref.long()), (N, K)
        assert torch.equal(out.cpu().long(), ref.long()), (N, K)
    pk.proxykv_destroy(ctx)


def _topk_with_patience(scores, K, patience):
    """The library's own launch of a Top-K, whose workgroups wait `patience` ticks of 10 ns for the others of their row."""
    import ctypes
    import re
    import subprocess
    names = subprocess.run(["nm", "-D", "--defined-only", pk.LIB_PATH], capture_output=True, text=True, check=True).stdout
    launch = getattr(pk.load(), re.search(r"\S*11launch_topkE\S*", names)[0])
    launch.argtypes = [ctypes.c_void_p] + [ctypes.c_int64] * 3 + [ctypes.c_void_p] * 2 + [ctypes.c_size_t, ctypes.c_void_p, ctypes.c_ulonglong]
    rows, N = scores.shape
    idx = torch.full((rows, K), -1, dtype=torch.int32, device="cuda")
    scratch = torch.full((1 << 22,), 7, dtype=torch.int32, device="cuda")
    assert launch(scores.data_ptr(), rows, N, K, idx.data_ptr(), scratch.data_ptr(), scratch.numel() * 4,
                  torch.cuda.current_stream().cuda_stream, patience) == 0
    torch.cuda.synchronize()
    return idx.cpu()


@pytest.mark.parametrize("patience", [0, 100, 20000])
@pytest.mark.parametrize("rows,N", [(28, 36865), (29, 131073), (64, 98760), (85, 172033), (256, 86016), (32, 8 * 86016)])
def test_topk_of_rows_that_workgroups_share(rows, N, patience):
    """Rows cut into one part to eight whose workgroups meet after every digit (28 rows and more, parts that fit the chip at once); with no
    patience, or 1 us of it, workgroups select from the whole row by themselves at one digit or another.  Ties across parts, NaN, infinities."""
    g = torch.Generator().manual_seed(N)
    base = 0.1 * torch.randn(3, N, generator=g)
    base[1] = torch.round(base[1] * 30) / 30
    base[2, torch.rand(N, generator=g) < 0.7] = float("nan")
    base[2, ::11], base[2, 1::13], base[2, 2::17] = float("inf"), float("-inf"), -0.0
    scores = base.repeat((rows + 2) // 3, 1)[:rows].contiguous().cuda()
    for K in (1, N // 3, N - 1):
        ref = oracle.topk(base, K).repeat((rows + 2) // 3, 1)[:rows]
        assert torch.equal(_topk_with_patience(scores, K, patience).long(), ref.long()), (rows, N, K)


def test_compact_bit_exact():
    ctx = _ctx(synth.CASES["tiny"])
    g = torch.Generator().manual_seed(3)
    for (L, H, N, D, K) in [(2, 3, 700, 128, 211), (1, 2, 130, 64, 130), (1, 1, 9, 128, 1), (1, 2, 300, 256, 77), (2, 1, 257, 32, 100),
                            (1, 1, 100, 8, 33)]:
        kv = torch.randn(2, L, H, N, D, generator=g).to(torch.bfloat16)
        s = torch.randn(L * H, N, generator=g)
        idx = oracle.topk(s, K).view(L, H, K)
        k_out, v_out = pk.proxykv_compact(ctx, kv[0].cuda(), kv[1].cuda(), idx.cuda())
        torch.cuda.synchronize()
        assert torch.equal(k_out.cpu().view(torch.int16), oracle.compact(kv[0], idx).view(torch.int16))
        assert torch.equal(v_out.cpu().view(torch.int16), oracle.compact(kv[1], idx).view(torch.int16))


def test_compact_inplace_and_mask_bit_exact():
    """The cache as its own destination: tokens 0 .. K-1 equal the out-of-place gather, the rest is untouched;
    the byte mask marks exactly the kept tokens.  Dense kept sets (sources right behind destinations), K = N,
    K = 1, several chunks of 128 with a ragged last one, unaligned mask rows."""
    ctx = _ctx(synth.CASES["tiny"])
    g = torch.Generator().manual_seed(4)
    for (L, H, N, D, K) in [(2, 3, 700, 128, 211), (1, 2, 130, 64, 130), (1, 1, 9, 128, 1), (1, 2, 1000, 128, 999),
                            (2, 2, 1537, 128, 640), (1, 3, 333, 256, 129)]:
        kv = torch.randn(2, L, H, N, D, generator=g).to(torch.bfloat16)
        s = torch.randn(L * H, N, generator=g)
        idx = oracle.topk(s, K).view(L, H, K)
        k, v = kv[0].cuda(), kv[1].cuda()
        pk.proxykv_compact_inplace(ctx, k, v, idx.cuda())
        m = pk.proxykv_mask(ctx, idx.cuda(), N)
        torch.cuda.synchronize()
        for got, src in ((k, kv[0]), (v, kv[1])):
            assert torch.equal(got[..., :K, :].cpu().view(torch.int16), oracle.compact(src, idx).view(torch.int16)), (N, K)
            assert torch.equal(got[..., K:, :].cpu().view(torch.int16), src[..., K:, :].view(torch.int16)), (N, K)
        assert torch.equal(m.cpu(), oracle.mask(idx, N)), (N, K)


@pytest.mark.parametrize("rows", [10, 200])
def test_topk_of_long_rows_by_bits_and_by_keys(rows):
    """The last pass over a long row compares scores with the ends of the threshold's bin and leaves two bits each for the kernel that
    writes.  Rows whose bin holds infinities, NaN, both zeros or the numbers next to them, and rows with many scores in it, go
    another way; and with 200 rows proxykv_topk_static's scratch memory has no room for the bits."""
    N, K = 50001, 20000
    g = torch.Generator().manual_seed(71)
    x = torch.randn(10, N, generator=g)
    half = torch.rand(10, N, generator=g) < 0.55
    x[1][half[1]] = float("-inf")
    x[2][half[2]] = float("nan")
    x[3][half[3]] = float("inf")
    x[4] = torch.where(half[4], torch.tensor(-0.0), torch.tensor(0.0)) * 1.0
    x[4][::3] = -1e-45 * torch.randint(1, 500, (N,), generator=g)[::3]      # the largest numbers below zero
    x[5] = torch.randint(-300, 300, (N,), generator=g) * 1e-45              # around zero, all in two bins
    x[6] = 1.0 + torch.randint(0, 900, (N,), generator=g) * 2.0 ** -23       # all in one bin of the last digit
    x[7][half[7]] = float(x[7].kthvalue(N - K + 1)[0])                       # more scores at the threshold than are kept
    x[8] = -x[8].abs() * 3e38
    x[9] = x[9] * 1e-41
    d = x.repeat(rows // 10, 1).cuda()
    ref = oracle.topk(x, K).repeat(rows // 10, 1)
    ctx = pk.proxykv_create(pk.config_for_case(synth.CASES["tiny"]))
    assert torch.equal(pk.proxykv_topk(ctx, d, K).cpu(), ref)
    out = torch.empty(rows, K, dtype=torch.int32, device="cuda")
    pk.proxykv_topk_static(ctx, d, K, out)
    torch.cuda.synchronize()
    assert torch.equal(out.cpu(), ref)
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("D", [8, 24, 40, 64, 72, 136, 256])
def test_compact_inplace_at_the_edges_of_chunks(D):
    """Kept counts around whole chunks of 128 tokens, every number of 16-byte pieces per thread, tokens with and without 128-byte
    parts, and kept tokens that each move by a few places only, so that a token's new place is another's old one."""
    _check_compact_inplace(D, 3, (1, 127, 128, 129, 255, 256, 257, 1000))


@pytest.mark.parametrize("D", [128, 256])
@pytest.mark.parametrize("rows", [255, 256])
def test_compact_inplace_at_the_edges_of_chunks_of_many_rows(D, rows):
    """The same where a workgroup's part of a token becomes 256 bytes instead of 128: from 256 rows and 513 kept tokens on."""
    _check_compact_inplace(D, rows, (1, 128, 257, 512, 513, 639, 640, 641))


@pytest.mark.parametrize("D,rows,counts", [(128, 3, (1919, 1920, 1921, 2560, 3201)), (128, 256, (960, 1281)), (256, 2, (959, 960, 961, 2000)),
                                           (72, 2, (3411, 3412, 4549)), (8, 1, (30720, 30721)), (64, 256, (1919, 1920, 1921))])
def test_compact_inplace_in_parts_of_a_row(D, rows, counts):
    """Rows long enough for several workgroups: a part takes 10 240 pieces of 16 bytes (640 tokens at D = 128, 1137 and seven pieces over at D = 72);
    kept counts at the line and around whole parts."""
    _check_compact_inplace(D, rows, counts)


def test_compact_inplace_in_parts_that_pay():
    """D = 256, 320 tokens to a part: six parts, one token less and one more, and eight; many rows whose third part is a third full."""
    _check_compact_inplace(256, 2, (1919, 1920, 1921, 2241))
    _check_compact_inplace(128, 256, (1500,))


def test_pooled_compaction_in_parts_of_more_heads_than_a_wave_has_lanes():
    """A layer's parts are dealt to its heads 64 at a time: 70 and 130 heads, some of which keep nothing and some everything."""
    _check_pooled([(2, 70, 5000, 64, 4000), (1, 130, 4000, 128, 3000)], nothing=slice(None))


def test_compact_inplace_in_a_graph_and_in_a_context_without_memory():
    """A graph moves whole rows, with the caller's pointers alone, whether the context that captures has room for an eager call's counters or not."""
    g = torch.Generator().manual_seed(5)
    rows, N, K, D = 4, 5000, 3000, 128
    idx = torch.stack([torch.randperm(N, generator=g)[:K].sort().values for _ in range(rows)]).to(torch.int32).view(1, rows, K).cuda()
    src = torch.randn(2, 1, rows, N, D, generator=g).to(torch.bfloat16).cuda()
    want = torch.gather(src, 3, idx.long().unsqueeze(0).unsqueeze(4).expand(2, -1, -1, -1, D))
    for warm in (False, True):
        ctx = _ctx(synth.CASES["tiny"])
        if warm:
            pk.proxykv_compact_inplace(ctx, src[0].clone(), src[1].clone(), idx)
        kv = src.clone()
        torch.cuda.synchronize()
        stream = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            pk.proxykv_compact_inplace(ctx, kv[0], kv[1], idx)
        for _ in range(3):
            kv.copy_(src)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(kv[:, :, :, :K], want) and torch.equal(kv[:, :, :, K:], src[:, :, :, K:]), warm
        del graph
        pk.proxykv_destroy(ctx)


def test_graph_of_an_in_place_compaction_outlives_its_context():
    """Captured by a context that has counters, replayed after longer calls have made its workspace grow, and after it is destroyed, with other
    memory taken in between: the same tokens."""
    g = torch.Generator().manual_seed(6)
    rows, N, K, D = 3, 6000, 4000, 128
    idx = torch.stack([torch.randperm(N, generator=g)[:K].sort().values for _ in range(rows)]).to(torch.int32).view(1, rows, K).cuda()
    src = torch.randn(2, 1, rows, N, D, generator=g).to(torch.bfloat16).cuda()
    want = torch.gather(src, 3, idx.long().unsqueeze(0).unsqueeze(4).expand(2, -1, -1, -1, D))
    ctx = _ctx(synth.CASES["tiny"])
    pk.proxykv_compact_inplace(ctx, src[0].clone(), src[1].clone(), idx)
    kv = src.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pk.proxykv_compact_inplace(ctx, kv[0], kv[1], idx)
    taken = []
    for step in range(3):
        if step == 1:
            pk.proxykv_topk(ctx, torch.randn(1, 40, 300000, device="cuda"), 1000)
        if step == 2:
            pk.proxykv_destroy(ctx)
        taken.append(torch.full((1 << 22,), 255, dtype=torch.uint8, device="cuda"))
        kv.copy_(src)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(kv[:, :, :, :K], want) and torch.equal(kv[:, :, :, K:], src[:, :, :, K:]), step


def test_in_place_compactions_of_one_context_side_by_side():
    """Calls on two streams, made by two threads, and on the capturing thread's other stream while one is captured: caches of their own, so nothing orders
    the calls, and the kept tokens of each are its own."""
    import threading
    g = torch.Generator().manual_seed(8)
    N, D = 5000, 128
    ctx = _ctx(synth.CASES["tiny"])
    jobs = []
    for rows, K in ((40, 3000), (64, 2500)):
        idx = torch.stack([torch.randperm(N, generator=g)[:K].sort().values for _ in range(rows)]).to(torch.int32).view(1, rows, K).cuda()
        src = torch.randn(2, 1, rows, N, D, generator=g).to(torch.bfloat16).cuda()
        want = torch.gather(src, 3, idx.long().unsqueeze(0).unsqueeze(4).expand(2, -1, -1, -1, D))
        jobs.append((torch.cuda.Stream(), idx, src, want, [src.clone() for _ in range(6)]))
    torch.cuda.synchronize()

    def work(stream, idx, src, want, caches):
        with torch.cuda.stream(stream):
            for kv in caches:
                pk.proxykv_compact_inplace(ctx, kv[0], kv[1], idx)
    threads = [threading.Thread(target=work, args=job) for job in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for _, idx, src, want, caches in jobs:
        for kv in caches:
            assert torch.equal(kv[:, :, :, :idx.shape[2]], want) and torch.equal(kv[:, :, :, idx.shape[2]:], src[:, :, :, idx.shape[2]:])

    fresh = _ctx(synth.CASES["tiny"])  # has no counters yet
    (side, idx, src, want, _), captured, eager = jobs[0], jobs[0][2].clone(), jobs[0][2].clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pk.proxykv_compact_inplace(fresh, captured[0], captured[1], idx)
        with torch.cuda.stream(side):
            pk.proxykv_compact_inplace(fresh, eager[0], eager[1], idx)
    graph.replay()
    torch.cuda.synchronize()
    for kv in (captured, eager):
        assert torch.equal(kv[:, :, :, :idx.shape[2]], want)
    pk.proxykv_destroy(fresh)
    pk.proxykv_destroy(ctx)


def test_pooled_compaction_of_many_heads_in_parts():
    """More heads than a wave's lanes deal parts to, with heads that keep nothing and heads that keep all; budgets of several parts each."""
    _check_pooled([(2, 70, 2000, 64, 1900), (1, 130, 1500, 128, 1000), (3, 2, 4000, 128, 1500)], nothing=slice(None))


def _check_compact_inplace(D, rows, counts):
    ctx = _ctx(synth.CASES["tiny"])
    g = torch.Generator().manual_seed(D)
    for K in counts:
        N = K + 5
        idx = torch.stack([torch.randperm(N, generator=g)[:K].sort().values for _ in range(rows)]).to(torch.int32)
        kv = torch.randn(2, rows, N, D, generator=g).to(torch.bfloat16)
        k, v = kv[0].cuda(), kv[1].cuda()
        pk.proxykv_compact_inplace(ctx, k.view(1, rows, N, D), v.view(1, rows, N, D), idx.view(1, rows, K).cuda())
        torch.cuda.synchronize()
        for got, src in ((k, kv[0]), (v, kv[1])):
            want = src.clone()
            want[:, :K] = torch.gather(src, 1, idx.long().unsqueeze(2).expand(-1, -1, D))
            assert torch.equal(got.cpu().view(torch.int16), want.view(torch.int16)), (rows, K)
    pk.proxykv_destroy(ctx)


def test_pooled_counts_of_more_heads_than_a_launch_has_waves():
    """72 million (layer, head) pairs of one token each: every pair keeps its token, and the waves that count take several pairs."""
    layers, heads = 2000, 36000
    ctx = _ctx(synth.CASES["tiny"])
    flat, counts = pk.proxykv_topk_pooled(ctx, torch.zeros(layers, heads, 1, device="cuda"), 1)
    torch.cuda.synchronize()
    assert bool((counts == 1).all())
    assert bool((flat == torch.arange(heads, device="cuda", dtype=torch.int32)).all())
    pk.proxykv_destroy(ctx)


def test_pooled_budget_bit_exact():
    """One budget per layer shared by its heads: kept flat indices, per-head counts, and the ragged in-place
    compaction, against the oracle.  Covers short rows (register-resident selection) and long ones, heads that
    get nothing, a head that gets everything it has, ties across heads."""
    _check_pooled([(2, 4, 700, 128, 211), (1, 3, 130, 64, 130), (1, 1, 9, 128, 1), (3, 8, 6000, 128, 1800),
                   (1, 2, 1537, 256, 300), (2, 5, 333, 64, 7)])


@pytest.mark.parametrize("D", [128, 256])
def test_pooled_budget_of_many_rows_bit_exact(D):
    """The same with 256 (layer, head) pairs and more, whose tokens move in parts of 256 bytes; in every layer a head gets nothing."""
    _check_pooled([(64, 4, 300, D, 129), (90, 3, 133, D, 40)], nothing=slice(None))


def _check_pooled(cases, nothing=0):
    ctx = _ctx(synth.CASES["tiny"])
    g = torch.Generator().manual_seed(5)
    for (L, H, N, D, K) in cases:
        s = torch.randn(L, H, N, generator=g)
        s[0, 0] += 4.0                                  # head 0 of layer 0 takes as much as it can
        if H > 2:
            s[nothing, 2] -= 8.0                        # and head 2 gets nothing
        if L > 1:
            s[1] = torch.round(s[1] * 2) / 2            # ties across heads
        flat_ref, counts_ref = oracle.topk_pooled(s, K)
        flat, counts = pk.proxykv_topk_pooled(ctx, s.cuda(), K)
        torch.cuda.synchronize()
        assert torch.equal(flat.cpu(), flat_ref), (N, K)
        assert torch.equal(counts.cpu(), counts_ref), (N, K)
        assert H < 3 or H * K > (H - 1) * N or bool((counts_ref[nothing, 2] == 0).all())
        kv = torch.randn(2, L, H, N, D, generator=g).to(torch.bfloat16)
        k, v = kv[0].cuda(), kv[1].cuda()
        pk.proxykv_compact_pooled(ctx, k, v, flat, counts)
        torch.cuda.synchronize()
        for l in range(L):
            start = 0
            for h in range(H):
                c = int(counts_ref[l, h])
                tok = (flat_ref[l, start:start + c].to(torch.int64) - h * N)
                start += c
                for got, src in ((k, kv[0]), (v, kv[1])):
                    assert torch.equal(got[l, h, :c].cpu().view(torch.int16), src[l, h][tok].view(torch.int16)), (N, K, l, h)
                    assert torch.equal(got[l, h, c:].cpu().view(torch.int16), src[l, h, c:].view(torch.int16)), (N, K, l, h)


def test_prune_selection_and_gather_in_one_launch_equals_two_launches():
    """proxykv_prune with the Top-K kernel gathering the kept tokens itself (the default) against the same call with the
    two kernels one after the other: same bits, for rows one workgroup selects and for rows split over several."""
    for (N, keep) in ((700, 0.3), (40000, 0.25)):
        case = synth.scaled_case(synth.CASES["llama_8k"], name=f"fused_{N}", L_s=1, H_q=2, H_kv=1, d=64, L_l=2, H_l=3, N=N, N_q=64,
                                 chunk=64, n_planted=2)
        q, kc, kr = synth.make_proxy_qk(case, device="cuda")
        k_t, v_t = synth.make_target_kv(case, device="cuda")
        ctx = _ctx(case, synth.make_mapper_weights(case.H_kv, case.H_l))
        outs = []
        for on in (True, False):
            pk.proxykv_set_fused_select(ctx, on)
            k_out, v_out, idx, K = pk.proxykv_prune(ctx, q, kc, kr, case.chunk, keep, k_t, v_t)
            torch.cuda.synchronize()
            outs.append((idx.clone(), k_out.view(torch.int16).clone(), v_out.view(torch.int16).clone()))
        for a, b in zip(*outs):
            assert torch.equal(a, b), N
        assert torch.equal(outs[0][1].cpu(), oracle.compact(k_t.cpu(), outs[0][0].cpu()).view(torch.int16))
        pk.proxykv_destroy(ctx)


# ----------------------------------------------------------------------------------------------
# scoring
# ----------------------------------------------------------------------------------------------

SCORE_CASES = {
    # several key/query tiles, ragged tails, chunk boundaries that cut query blocks
    "d64_ragged": dict(L_s=2, H_q=4, H_kv=2, d=64, N=1000, N_q=700, chunk=300, n_planted=6),
    "d64_gqa7": dict(L_s=1, H_q=14, H_kv=2, d=64, N=1500, N_q=1500, chunk=512, n_planted=8),
    "d128": dict(L_s=2, H_q=6, H_kv=2, d=128, N=900, N_q=640, chunk=256, n_planted=6),
    "one_query": dict(L_s=1, H_q=1, H_kv=1, d=64, N=5, N_q=1, chunk=1, n_planted=0),
    "small_chunks": dict(L_s=1, H_q=2, H_kv=1, d=64, N=300, N_q=300, chunk=17, n_planted=3),
}


def _score_case(name):
    return synth.scaled_case(synth.CASES["llama_8k"], name=name, L_l=1, H_l=2, **SCORE_CASES[name])


@pytest.mark.parametrize("name", list(SCORE_CASES))
def test_score_matches_oracle(name):
    case = _score_case(name)
    q, kc, kr = synth.make_proxy_qk(case)
    ref = oracle.score(q.double(), kc.double(), kr.double(), case.chunk)
    ctx = _ctx(case)
    x = pk.proxykv_score(ctx, q.cuda(), kc.cuda(), kr.cuda(), case.chunk)
    torch.cuda.synchronize()
    assert_close(x, ref, f"score[{name}]")
    x_min, x_max = float(x.min()), float(x.max())
    assert x_min >= 0.0 and x_max <= 1.0, (x_min, x_max)


@pytest.mark.parametrize("name", list(SCORE_CASES))
def test_score_sum_form_matches_oracle(name):
    """reduce = SUM: the accumulation over the query axis that Sec. 3 prints, over all heads of the group."""
    case = _score_case(name)
    q, kc, kr = synth.make_proxy_qk(case)
    ref = oracle.score(q.double(), kc.double(), kr.double(), case.chunk, reduce="sum")
    cfg = pk.config_for_case(case)
    cfg.reduce = pk.PROXYKV_REDUCE_SUM
    ctx = pk.proxykv_create(cfg)
    x = pk.proxykv_score(ctx, q.cuda(), kc.cuda(), kr.cuda(), case.chunk)
    torch.cuda.synchronize()
    assert_close(x, ref, f"score sum[{name}]")
    # every query row spends at most all of its probability on the context keys
    assert float(x.sum(dim=-1).max()) <= case.G * case.N_q * (1.0 + 1e-5)


@pytest.mark.parametrize("name", list(SCORE_CASES))
def test_score_self_matches_oracle(name):
    """The feature as Sec. 3 prints it: causal self-attention of the sequence, summed over queries and group heads."""
    case = _score_case(name)
    q, _, k = synth.make_proxy_qk(case)                 # the reconstruction keys serve as the sequence's own keys
    ref = oracle.score_self(q.double(), k.double())
    ctx = _ctx(case)
    x = pk.proxykv_score_self(ctx, q.cuda(), k.cuda())
    torch.cuda.synchronize()
    assert_close(x, ref, f"score_self[{name}]")
    # every query row is a probability vector over its visible keys
    total = x.double().sum(dim=-1).cpu()
    assert torch.allclose(total, torch.full_like(total, float(case.G * case.N_q)), rtol=1e-4)


def test_score_self_fp32_inputs_and_block_boundaries():
    """fp32 inputs are rounded to bf16 on entry; lengths at and around the 256-key / 128-query tile sizes."""
    base = synth.scaled_case(synth.CASES["llama_8k"], name="self_f32", L_s=1, H_q=2, H_kv=1, d=64, L_l=1, H_l=2, N=8, N_q=8, chunk=8,
                             n_planted=0)
    ctx = _ctx(base)
    for N in (1, 2, 127, 128, 129, 255, 256, 257, 513):
        g = torch.Generator().manual_seed(N)
        q = torch.randn(1, 2, N, 64, generator=g)
        k = torch.randn(1, 1, N, 64, generator=g)
        ref = oracle.score_self(q, k)                   # the oracle rounds to bf16 itself
        x = pk.proxykv_score_self(ctx, q.cuda(), k.cuda())
        torch.cuda.synchronize()
        assert_close(x, ref, f"score_self fp32 N={N}")


@pytest.mark.parametrize("N,N_q,chunk", [(1, 1, 1), (1, 300, 100), (129, 1, 5), (2, 130, 1000), (513, 257, 256)])
def test_score_degenerate_shapes(N, N_q, chunk):
    """One context key, one query, a chunk longer than the query axis, lengths one past the tile sizes; max and sum forms."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name=f"deg_{N}_{N_q}", L_s=1, H_q=4, H_kv=2, d=64, L_l=1, H_l=2, N=N, N_q=N_q,
                             chunk=chunk, n_planted=0)
    q, kc, kr = synth.make_proxy_qk(case)
    for reduce, code in (("max", pk.PROXYKV_REDUCE_MAX), ("sum", pk.PROXYKV_REDUCE_SUM)):
        cfg = pk.config_for_case(case)
        cfg.reduce = code
        ctx = pk.proxykv_create(cfg)
        x = pk.proxykv_score(ctx, q.cuda(), kc.cuda(), kr.cuda(), chunk)
        torch.cuda.synchronize()
        assert_close(x, oracle.score(q.double(), kc.double(), kr.double(), chunk, reduce=reduce), f"score {reduce} N={N} N_q={N_q}")
        pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("L,H_q,H_kv", [(1, 1, 1), (3, 2, 1), (9, 1, 1), (13, 2, 1), (4, 4, 4)])
@pytest.mark.parametrize("N", [257, 1100])
def test_score_of_groups_that_do_not_fill_the_xcds_evenly(L, H_q, H_kv, N):
    """Pass 2 deals the groups' key blocks to eight XCDs: one group, three, nine, thirteen (and sixteen, two each); max, sum and causal forms."""
    g = torch.Generator().manual_seed(L + N)
    q = torch.randn(L, H_q, 300, 64, generator=g).bfloat16()
    kc, kr = (torch.randn(L, H_kv, n, 64, generator=g).bfloat16() for n in (N, 300))
    own = torch.randn(L, H_q, N, 64, generator=g).bfloat16()
    for reduce, code in (("max", pk.PROXYKV_REDUCE_MAX), ("sum", pk.PROXYKV_REDUCE_SUM)):
        cfg = pk.make_config(L, H_q, H_kv, 64, 1, 4, 128)
        cfg.reduce = code
        ctx = pk.proxykv_create(cfg)
        x = pk.proxykv_score(ctx, q.cuda(), kc.cuda(), kr.cuda(), 128)
        xs = pk.proxykv_score_self(ctx, own.cuda(), kc.cuda())
        torch.cuda.synchronize()
        assert_close(x, oracle.score(q, kc, kr, 128, reduce=reduce), f"score {reduce}")
        assert_close(xs, oracle.score_self(own, kc), "score_self")
        pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("N,N_q,chunk", [(1, 1, 1), (130, 257, 100), (700, 300, 128), (1000, 1000, 2048), (4096, 70, 64), (4097, 70, 64)])
def test_score_of_fp32_inputs_is_that_of_their_bf16_roundings(N, N_q, chunk):
    """Up to 4096 keys, where workgroups share a block's, pass 1 rounds fp32 inputs itself and leaves the copies that pass 2 reads; max, sum and
    causal forms, groups of two heads, ties of the rounding and large values among the inputs."""
    g = torch.Generator().manual_seed(N)
    q, kc, kr, own = (torch.randn(2, h, n, 64, generator=g) for h, n in ((4, N_q), (2, N), (2, N_q), (4, N)))
    q[0, 0, 0, :8] = torch.tensor([1.00390625, 1.01171875, -1.00390625, 3e-39, 1e-45, -0.0, 2.5e4, -2.5e4])
    for reduce in (pk.PROXYKV_REDUCE_MAX, pk.PROXYKV_REDUCE_SUM):
        cfg = pk.make_config(2, 4, 2, 64, 1, 4, 128)
        cfg.reduce = reduce
        ctx = pk.proxykv_create(cfg)
        wide, half = ([t.to(dtype).cuda() for t in (q, kc, kr, own)] for dtype in (torch.float32, torch.bfloat16))
        got = [pk.proxykv_score(ctx, t[0], t[1], t[2], chunk) for t in (wide, half)] + [pk.proxykv_score_self(ctx, t[3], t[1]) for t in (wide, half)]
        torch.cuda.synchronize()
        assert torch.equal(got[0], got[1]) and torch.equal(got[2], got[3])
        pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("d,N,N_q,chunk", [(64, 1, 3, 2), (64, 700, 257, 100), (64, 1030, 130, 64), (128, 65, 300, 1000), (128, 900, 64, 33),
                                          (128, 1100, 200, 256), (64, 2600, 1700, 512)])
def test_score_few_and_many_query_blocks_agree(d, N, N_q, chunk):
    """Few query blocks: several workgroups share a block's keys (and, in the max form, a key block's queries); many: one
    workgroup each, or a few where the last turn on the chip would be half empty (the last two shapes).  The same layer alone and as one of 192 must agree to the rounding of 32-bit sums and exponentials
    (log-sum-exps up to about 2^4, whose last bit is 1e-6, scaled back: 2e-5), and both with the oracle."""
    L, H_q, H_kv = 192, 4, 2
    g = torch.Generator().manual_seed(N + N_q)
    q = torch.randn(L, H_q, N_q, d, generator=g).bfloat16()
    kc = torch.randn(L, H_kv, N, d, generator=g).bfloat16()
    kr = torch.randn(L, H_kv, N_q, d, generator=g).bfloat16()
    for reduce in (pk.PROXYKV_REDUCE_MAX, pk.PROXYKV_REDUCE_SUM):
        many, few = (pk.make_config(n, H_q, H_kv, d, 1, 4, 128) for n in (L, 1))
        many.reduce = few.reduce = reduce
        cm, cf = pk.proxykv_create(many), pk.proxykv_create(few)
        x = pk.proxykv_score(cm, q.cuda(), kc.cuda(), kr.cuda(), chunk)
        xs = pk.proxykv_score_self(cm, q.cuda(), kr.cuda())
        for l in (0, L - 1):
            one = [t[l:l + 1].contiguous() for t in (q, kc, kr)]
            y = pk.proxykv_score(cf, *(t.cuda() for t in one), chunk)
            ys = pk.proxykv_score_self(cf, one[0].cuda(), one[2].cuda())
            torch.cuda.synchronize()
            torch.testing.assert_close(y.cpu(), x[l:l + 1].cpu(), rtol=2e-5, atol=1e-9)
            torch.testing.assert_close(ys.cpu(), xs[l:l + 1].cpu(), rtol=2e-5, atol=1e-9)
            assert_close(y, oracle.score(*one, chunk, reduce="max" if reduce == pk.PROXYKV_REDUCE_MAX else "sum"), f"score layer {l}")
            assert_close(ys, oracle.score_self(one[0], one[2]), f"score_self layer {l}")
        pk.proxykv_destroy(cm)
        pk.proxykv_destroy(cf)


@pytest.mark.parametrize("N_q", [256, 257])
@pytest.mark.parametrize("scale", [1.0, 30.0])
def test_score_of_few_query_blocks_and_of_more(N_q, scale):
    """47 layers of 8 heads of 128: 256 queries make 376 blocks of pass 1, whose keys workgroups share; 257 make 752, one workgroup each.  Also
    with nearly one-hot rows, where its reference is replaced many times."""
    _score_47_layers(N_q, 300, scale)


@pytest.mark.parametrize("N", [1394, 1395])
@pytest.mark.parametrize("scale", [1.0, 30.0])
def test_score_where_the_wide_tiles_end(N, scale):
    """752 blocks, one workgroup each: up to 2^20 blocks times keys with 32-column matrix tiles, beyond it with 16-column ones."""
    _score_47_layers(257, N, scale)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N_q", [769, 1024, 1025, 2048])
def test_score_of_heads_of_four_and_eight_query_blocks(N_q, d):
    """Four and eight query blocks per head, whose order is turned from head to head, and five, whose order is not."""
    _score_47_layers(N_q, 300, 1.0, d)


@pytest.mark.parametrize("N", [1395, 1536])
def test_score_of_whole_tiles_out_of_range(N):
    """Heads of 64 in blocks of their own, logits of a standard deviation of 30: a column's sum leaves its range in many whole tiles, which are undone and
    summed again with new references."""
    _score_47_layers(257, N, 30.0, 64)


@pytest.mark.parametrize("far", [11.0, 40.0])
def test_score_of_keys_far_above_the_reference_in_a_middle_tile(far):
    """Context keys that are `far` times a query, from the fourth tile on, in two tiles in a row and in the last whole one, and reconstruction keys like that in a
    tile that every query of a block sees: the sum of a tile, begun while the one before was summed, exceeds 2^100 (11: about 2^127) or is infinite.
    Max and sum forms; heads of 64, blocks of their own."""
    L, H_q, H_kv, N_q, N, chunk = 48, 8, 2, 400, 1340, 300
    g = torch.Generator().manual_seed(int(far))
    q = torch.randn(L, H_q, N_q, 64, generator=g).bfloat16()
    kc, kr = (torch.randn(L, H_kv, n, 64, generator=g).bfloat16() for n in (N, N_q))
    for l in range(L):
        for h in range(H_kv):
            for at in (400, 530, 650, 1279) if l % 3 else (900, 901, 1024, 1339):
                i = int(torch.randint(N_q, (1,), generator=g))
                kc[l, h, at] = (far * q[l, 4 * h + (at + l) % 4, i].float()).bfloat16()
            if l % 2:  # seen by the queries behind it in its chunk
                kr[l, h, 130] = (far * q[l, 4 * h, 299].float()).bfloat16()
    for reduce, code in (("max", pk.PROXYKV_REDUCE_MAX), ("sum", pk.PROXYKV_REDUCE_SUM)):
        cfg = pk.make_config(L, H_q, H_kv, 64, 1, 4, 128)
        cfg.reduce = code
        ctx = pk.proxykv_create(cfg)
        x = pk.proxykv_score(ctx, q.cuda(), kc.cuda(), kr.cuda(), chunk)
        torch.cuda.synchronize()
        assert_close(x, oracle.score(q, kc, kr, chunk, reduce=reduce), f"score {reduce}")
        pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("far", [0.0, 11.0, 40.0])
def test_causal_score_of_keys_far_above_the_reference(far):
    """The causal form beyond 2048 tokens, whose whole tiles are the reconstruction's: the same for keys in the middle of the sequence, at its end and in its
    first tile."""
    L, H_q, H_kv, N = 6, 8, 2, 2222
    g = torch.Generator().manual_seed(3)
    q = torch.randn(L, H_q, N, 64, generator=g).bfloat16()
    k = torch.randn(L, H_kv, N, 64, generator=g).bfloat16()
    if far:
        for l in range(L):
            for h in range(H_kv):
                for at in (700, 831, 1500, 2100) if l % 2 else (40, 1000, 1001, 2047):
                    k[l, h, at] = (far * q[l, 4 * h + at % 4, int(torch.randint(at, N, (1,), generator=g))].float()).bfloat16()
    ctx = pk.proxykv_create(pk.make_config(L, H_q, H_kv, 64, 1, 4, 128))
    x = pk.proxykv_score_self(ctx, q.cuda(), k.cuda())
    torch.cuda.synchronize()
    assert_close(x, oracle.score_self(q, k), "score_self")
    pk.proxykv_destroy(ctx)


def _score_47_layers(N_q, N, scale, d=128):
    L, H_q, H_kv, chunk = 47, 8, 2, 200
    g = torch.Generator().manual_seed(N_q)
    q = (scale * torch.randn(L, H_q, N_q, d, generator=g)).bfloat16()
    kc, kr = (torch.randn(L, H_kv, n, d, generator=g).bfloat16() for n in (N, N_q))
    ctx = pk.proxykv_create(pk.make_config(L, H_q, H_kv, d, 1, 4, 128))
    x = pk.proxykv_score(ctx, q.cuda(), kc.cuda(), kr.cuda(), chunk)
    torch.cuda.synchronize()
    for l in (0, L - 1):
        assert_close(x[l:l + 1], oracle.score(q[l:l + 1], kc[l:l + 1], kr[l:l + 1], chunk), f"score layer {l}")
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("scale", [8.0, 30.0])
def test_score_large_logits(scale):
    """Inputs scaled up until the softmax rows are nearly one-hot (logits of several hundred): the running reference of
    pass 1 is replaced many times, probabilities are either about one or far below the absolute tolerance."""
    case = _score_case("d64_ragged")
    q, kc, kr = synth.make_proxy_qk(case)
    q, kc, kr = (q.float() * scale).to(torch.bfloat16), (kc.float() * scale).to(torch.bfloat16), (kr.float() * scale).to(torch.bfloat16)
    for reduce, code in (("max", pk.PROXYKV_REDUCE_MAX), ("sum", pk.PROXYKV_REDUCE_SUM)):
        cfg = pk.config_for_case(case)
        cfg.reduce = code
        ctx = pk.proxykv_create(cfg)
        x = pk.proxykv_score(ctx, q.cuda(), kc.cuda(), kr.cuda(), case.chunk)
        torch.cuda.synchronize()
        assert_close(x, oracle.score(q.double(), kc.double(), kr.double(), case.chunk, reduce=reduce), f"score {reduce} x{scale}")
        pk.proxykv_destroy(ctx)
    xs = pk.proxykv_score_self(_ctx(case), q.cuda(), kr.cuda())
    torch.cuda.synchronize()
    assert_close(xs, oracle.score_self(q.double(), kr.double()), f"score_self x{scale}")


def test_score_tiny_case_fp32_inputs_and_planted_keys():
    case = synth.CASES["tiny"]
    q, kc, kr = synth.make_proxy_qk(case)
    assert q.dtype == torch.float32
    ref = oracle.score(q, kc, kr, case.chunk)          # the oracle rounds the inputs to bf16 itself
    ctx = _ctx(case)
    x = pk.proxykv_score(ctx, q.cuda(), kc.cuda(), kr.cuda(), case.chunk)
    torch.cuda.synchronize()
    assert_close(x, ref, "score[tiny]")
    plan = synth.plant_plan(case)
    K = pk.proxykv_keep_count(case.N, 0.3)
    kept = pk.proxykv_topk(ctx, x, K).cpu()
    for l in range(case.L_s):
        for h in range(case.H_kv):
            assert set(plan["pos"][l, h].tolist()) <= set(kept[l, h].tolist())
            assert bool((x[l, h].cpu()[plan["pos"][l, h]] > 0.5).all())


def test_score_uniform_rows_closed_form():
    """Zero queries: every row is uniform and the score is exactly 1/(N+1)."""
    case = synth.scaled_case(_score_case("d64_ragged"), n_planted=0)
    q, kc, kr = synth.make_proxy_qk(case)
    ctx = _ctx(case)
    x = pk.proxykv_score(ctx, torch.zeros_like(q).cuda(), kc.cuda(), kr.cuda(), case.chunk)
    torch.cuda.synchronize()
    torch.testing.assert_close(x.cpu(), torch.full_like(x.cpu(), 1.0 / (case.N + 1)), rtol=1e-5, atol=0)


# ----------------------------------------------------------------------------------------------
# mapper
# ----------------------------------------------------------------------------------------------

MAP_CASES = {
    "one_window": dict(L_s=1, H_kv=2, H_q=4, L_l=1, H_l=4, N=512),
    "two_windows_ragged": dict(L_s=2, H_kv=8, H_q=8, L_l=3, H_l=8, N=2500),
    "three_windows_short_tail": dict(L_s=1, H_kv=2, H_q=2, L_l=2, H_l=4, N=3100),
}


@pytest.mark.parametrize("name", list(MAP_CASES))
def test_mapper_matches_oracle(name):
    case = synth.scaled_case(synth.CASES["llama_8k"], name=name, N_q=64, chunk=64, n_planted=0, **MAP_CASES[name])
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(17)
    # score-like input: mostly small positive values with a few near one
    X = torch.rand(case.L_s, case.H_kv, case.N, generator=g) ** 8
    X = X.to(torch.float32)
    ref = oracle.mapper(X, w, case.L_l)
    ctx = _ctx(case, w)
    y = pk.proxykv_map(ctx, X.cuda())
    torch.cuda.synchronize()
    assert_close(y, ref, f"map[{name}]")
    pairing = pk.proxykv_layer_pairing(ctx.cfg)
    for a in range(case.L_l):
        for b in range(a + 1, case.L_l):
            if pairing[a] == pairing[b]:
                assert torch.equal(y[a], y[b])


@pytest.mark.parametrize("N", [1, 2, 65, 2049])
def test_mapper_degenerate_lengths(N):
    """One token, two tokens, just over one MFMA key tile, and one token past the first window (a second window of 1025)."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name=f"len{N}", L_s=2, H_kv=2, H_q=2, L_l=2, H_l=4, N=N, N_q=1, chunk=1,
                             n_planted=0)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(100 + N)
    X = (torch.rand(case.L_s, case.H_kv, N, generator=g) ** 8).to(torch.float32)
    ctx = _ctx(case, w)
    y = pk.proxykv_map(ctx, X.cuda())
    torch.cuda.synchronize()
    assert_close(y, oracle.mapper(X, w, case.L_l), f"map N={N}")
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("L_s,L_l,N", [(33, 33, 5), (5, 3, 257), (3, 3, 2305), (4, 9, 255)])
def test_mapper_batches_of_layers(L_s, L_l, N):
    """Distinct proxy layers share their launches: more layers than one batch takes, layers that no target layer reads,
    several target layers per proxy layer, lengths just past and just short of the 256-row stride between two layers, and
    a second window.  Scores differ by a factor between layers, so a row that leaked into a neighbour would show."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="batch", L_s=L_s, H_kv=2, H_q=2, L_l=L_l, H_l=4, N=N, N_q=1, chunk=1,
                             n_planted=0)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(300 + N)
    X = (torch.rand(L_s, case.H_kv, N, generator=g) ** 8) * (1.0 + torch.arange(L_s).view(-1, 1, 1) % 7)
    ctx = _ctx(case, w)
    y = pk.proxykv_map(ctx, X.float().cuda())
    torch.cuda.synchronize()
    assert_close(y, oracle.mapper(X.float(), w, L_l), f"map {L_s} -> {L_l} layers, N={N}")
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("L,N", [(1, 2049), (1, 2500), (1, 3072), (1, 3073), (2, 2048), (2, 2049), (3, 1365), (3, 1366)])
def test_mapper_of_few_rows_in_large_tiles(L, N):
    """Just more rows than the small-tile kernels take: one layer of two and three windows (overlap averaging, a token's row stored
    into both windows), two and three layers of one window and of two."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="small", L_s=L, H_kv=2, H_q=2, L_l=L, H_l=4, N=N, N_q=1, chunk=1,
                             n_planted=0)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(400 + N)
    X = (torch.rand(L, case.H_kv, N, generator=g) ** 8) * (1.0 + torch.arange(L).view(-1, 1, 1))
    ctx = _ctx(case, w)
    y = pk.proxykv_map(ctx, X.float().cuda())
    torch.cuda.synchronize()
    assert_close(y, oracle.mapper(X.float(), w, L), f"map {L} layers, N={N}")
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("L,N", [(32, 129), (26, 191), (2, 2175), (2, 2176), (2, 2177), (1, 4096)])
def test_mapper_at_the_edges_of_a_block(L, N):
    """The large tiles take blocks of 128 rows: one row in a layer's last block, all but one, a whole one, keys that end inside and at the
    end of an attention tile of 64, layers of several blocks side by side, a last window of whole blocks."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="block", L_s=L, H_kv=2, H_q=2, L_l=L, H_l=4, N=N, N_q=1, chunk=1,
                             n_planted=0)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(600 + N)
    X = (torch.rand(L, case.H_kv, N, generator=g) ** 8) * (1.0 + torch.arange(L).view(-1, 1, 1) % 7)
    ctx = _ctx(case, w)
    y = pk.proxykv_map(ctx, X.float().cuda())
    torch.cuda.synchronize()
    assert_close(y, oracle.mapper(X.float(), w, L), f"map {L} layers, N={N}")
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("N", [2561, 2688, 2689, 2816])
def test_mapper_products_in_tiles_of_128_and_of_256_rows_agree(N):
    """One layer's projection has at most 44 large tiles and takes tiles of 128 rows, as the convolution always does; that of eight layers has
    352 and takes the large ones.  Layers whose last tile holds one row, or all, of 128, alone and among 16: the same bits.  Tokens of
    a third window, whose rows go to two windows."""
    case = lambda L: synth.scaled_case(synth.CASES["llama_8k"], name="tiles", L_s=L, H_kv=8, H_q=8, L_l=L, H_l=3, N=N, N_q=1, chunk=1, n_planted=0)
    w = synth.make_mapper_weights(8, 3)
    X, y = torch.rand(16, 8, N, generator=torch.Generator().manual_seed(N)) ** 8, []
    for L in (1, 16):
        ctx = _ctx(case(L), w)
        y.append(pk.proxykv_map(ctx, X[:L].float().contiguous().cuda())[0].cpu())
        torch.cuda.synchronize()
        pk.proxykv_destroy(ctx)
    assert torch.equal(y[0], y[1])
    assert_close(y[0][None], oracle.mapper(X[:1].float(), w, 1), f"map 1 layer, N={N}")


@pytest.mark.parametrize("few,many,N", [(4, 24, 1000), (4, 24, 961), (2, 16, 2303), (2, 16, 3072)])
def test_mapper_attention_of_128_and_of_256_queries_agree(few, many, N):
    """The attention of few layers, at most 256 workgroups of 256 queries, is given to twice as many; that of many layers is not.  A
    window's queries end in a workgroup's first wave, or its last; the same bits either way."""
    case = lambda L: synth.scaled_case(synth.CASES["llama_8k"], name="queries", L_s=L, H_kv=2, H_q=2, L_l=L, H_l=4, N=N, N_q=1, chunk=1, n_planted=0)
    w = synth.make_mapper_weights(2, 4)
    X, y = torch.rand(many, 2, N, generator=torch.Generator().manual_seed(N)) ** 8, []
    for L in (few, many):
        ctx = _ctx(case(L), w)
        y.append(pk.proxykv_map(ctx, X[:L].float().contiguous().cuda())[:few].cpu())
        torch.cuda.synchronize()
        pk.proxykv_destroy(ctx)
    assert torch.equal(y[0], y[1])
    assert_close(y[0][:1], oracle.mapper(X[:few].float(), w, few, layers=[0])[:1], f"map {few} layers, N={N}")


@pytest.mark.parametrize("L,N", [(1, 2048), (2, 1280), (2, 1281), (5, 512), (5, 513), (20, 65), (21, 65)])
def test_mapper_where_the_small_tiles_end(L, N):
    """40 tiles of 64 rows are the last that the small tiles take: on the line and one row or layer beyond it, where half blocks begin."""
    test_mapper_at_the_edges_of_a_block(L, N)


@pytest.mark.parametrize("d_ffn,c_mid,n_enc", [(256, 256, 1), (512, 512, 2), (4096, 768, 1), (2048, 256, 0)])
@pytest.mark.parametrize("L,N", [(2, 300), (2, 2600), (33, 1030)])
def test_mapper_of_other_sizes(d_ffn, c_mid, n_enc, L, N):
    """One chunk of hidden features and sixteen, a wider stem, encoders of no, one and two layers (whose first launch is followed by the
    last); small tiles, half blocks of three windows and whole blocks, in more layers than one batch takes."""
    dims = synth.MapperDims(d_ffn=d_ffn, c_mid=c_mid, n_enc_layers=n_enc)
    w = synth.make_mapper_weights(2, 3, dims)
    ctx = pk.proxykv_create(pk.make_config(L, 2, 2, 64, L, 3, 128, d_ffn=d_ffn, c_mid=c_mid, n_enc_layers=n_enc))
    pk.proxykv_set_mapper_weights(ctx, w)
    X = torch.rand(L, 2, N, generator=torch.Generator().manual_seed(N)) ** 8
    y = pk.proxykv_map(ctx, X.cuda()).cpu()
    torch.cuda.synchronize()
    for l in {0, L - 1}:
        assert_close(y[l:l + 1], oracle.mapper(X, w, L, layers=[l])[l:l + 1], f"map d_ffn={d_ffn} c_mid={c_mid} {n_enc} layers, N={N}, layer {l}")
    pk.proxykv_destroy(ctx)


def test_mapper_half_blocks_are_whole_blocks_bit_for_bit():
    """40 layers of 600 tokens are two times 100 blocks in two lanes, more than these run as halves; the first 8 of them alone are 40 blocks in one
    lane, which run as halves, of which each layer's last holds 24 rows."""
    y = []
    for L in (40, 8):
        case = synth.scaled_case(synth.CASES["llama_8k"], name="halves", L_s=L, H_kv=2, H_q=2, L_l=L, H_l=4, N=600, N_q=1, chunk=1, n_planted=0)
        w = synth.make_mapper_weights(case.H_kv, case.H_l)
        X = (torch.rand(40, case.H_kv, 600, generator=torch.Generator().manual_seed(77)) ** 8)[:L].contiguous()
        ctx = _ctx(case, w)
        y.append(pk.proxykv_map(ctx, X.float().cuda())[:8].clone())
        torch.cuda.synchronize()
        pk.proxykv_destroy(ctx)
    assert torch.equal(y[0], y[1])


@pytest.mark.parametrize("N,halves,wholes", [(1024, 24, 26), (1025, 20, 22), (600, 38, 40)])
def test_mapper_half_blocks_of_two_lanes_are_whole_blocks_bit_for_bit(N, halves, wholes):
    """Two lanes' blocks run as halves up to three quarters of the CUs, 192 of both lanes: layers that make so many, or the next fewer, against
    the same layers among more.  The halves are compared with the oracle as well."""
    X, y = torch.rand(wholes, 2, N, generator=torch.Generator().manual_seed(N)) ** 8, []
    w = synth.make_mapper_weights(2, 4)
    for L in (halves, wholes):
        case = synth.scaled_case(synth.CASES["llama_8k"], name="halves", L_s=L, H_kv=2, H_q=2, L_l=L, H_l=4, N=N, N_q=1, chunk=1, n_planted=0)
        ctx = _ctx(case, w)
        y.append(pk.proxykv_map(ctx, X[:L].float().contiguous().cuda())[:halves].cpu())
        torch.cuda.synchronize()
        pk.proxykv_destroy(ctx)
    assert torch.equal(y[0], y[1])
    for l in (0, halves - 1):
        assert_close(y[0][l:l + 1], oracle.mapper(X[:halves].float(), w, halves, layers=[l])[l:l + 1], f"map {halves} layers, N={N}, layer {l}")


def test_mapper_with_scores_beyond_the_half_range():
    """Sum-form scores with an attention sink (Sec. 3 prints the feature as a sum over the query axis, so one key can
    collect a share of every row): the first conv block's output reaches 1.4e5, beyond what IEEE half holds.  The
    library stores that operand as a half value times a power of two taken from the layer's largest score; the oracle
    rounds it to an 11-bit significand without a range limit.  Also the same mapper on ordinary scores right after
    (the range exponent is per call and per layer)."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="sink", L_s=2, H_kv=2, H_q=2, L_l=2, H_l=4, N=700, N_q=1, chunk=1,
                             n_planted=0)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(5)
    X = (torch.rand(case.L_s, case.H_kv, case.N, generator=g) * 8).to(torch.float32)
    X[0, :, 0] = 1.0e5                                   # layer 0: a sink at the first token and a smaller one mid-way
    X[0, :, 350] = 3.0e4
    ref = oracle.mapper(X, w, case.L_l)
    assert bool(torch.isfinite(ref).all())
    a1 = torch.nn.functional.conv1d(X[0:1].double(), w["stem.conv1.weight"].double(), w["stem.conv1.bias"].double(), padding=1)
    assert float(a1.abs().max()) > 65504.0                # the case does leave half's range
    ctx = _ctx(case, w)
    y = pk.proxykv_map(ctx, X.cuda())
    torch.cuda.synchronize()
    assert_close(y, ref, "map with a sink")
    X2 = (torch.rand(case.L_s, case.H_kv, case.N, generator=g) ** 8).to(torch.float32)
    y2 = pk.proxykv_map(ctx, X2.cuda())
    torch.cuda.synchronize()
    assert_close(y2, oracle.mapper(X2, w, case.L_l), "map after a sink")
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("sink", [30.0, 300.0, 3.0e3])
def test_mapper_with_logits_far_above_those_of_the_first_keys(sink):
    """The window attention of the large tiles takes a query's reference from its first 64 keys and raises it where a later logit is
    more than 2^8 times as likely.  Sinks behind the first keys of both windows give logits in the thousands; a cut last tile, two
    layers of which one is ordinary.  Three seeds and two ways of summing stay within 0.29 of the bound up to 3e3; at 3e4 logits reach the millions, where one rounding of an operand
    to half decides between two keys, and both ways are the same 4.9e-3 off."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="late", L_s=2, H_kv=2, H_q=2, L_l=2, H_l=4, N=2200, N_q=1, chunk=1, n_planted=0)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(8)
    X = (torch.rand(case.L_s, case.H_kv, case.N, generator=g) ** 8).to(torch.float32)
    X[0, :, 700] = sink
    X[0, :, 1900] = 0.3 * sink
    X[0, :, 2199] = 0.1 * sink
    ctx = _ctx(case, w)
    y = pk.proxykv_map(ctx, X.cuda())
    torch.cuda.synchronize()
    assert_close(y, oracle.mapper(X, w, case.L_l), f"map with late sinks of {sink:g}")
    pk.proxykv_destroy(ctx)


def test_mapper_takes_no_longer_where_the_attention_is_sharp():
    """Attention weights that go beyond what half holds relative to the first keys' (here in every workgroup: q and k five times as
    wide) cost a rescaling each and not another pass over the keys, which made this 1.42 times as long."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="sharp", L_s=8, H_kv=2, H_q=2, L_l=8, H_l=4, N=8192, N_q=1, chunk=1, n_planted=0)
    X = (torch.rand(case.L_s, case.H_kv, case.N, generator=torch.Generator().manual_seed(9)) ** 8).cuda()
    ctxs = []
    for width in (1.0, 5.0):
        w = synth.make_mapper_weights(case.H_kv, case.H_l)
        for name in w:
            if name.endswith("in_proj.weight"):
                w[name] = torch.cat([w[name][:1024] * width, w[name][1024:]])
        ctxs.append(_ctx(case, w))
    best = [float("inf")] * 2
    y = torch.empty(case.L_l, case.H_l, case.N, device="cuda")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for rep in range(6):
        for i, ctx in enumerate(ctxs):
            a.record()
            for _ in range(4):
                pk.proxykv_map(ctx, X, yhat=y)
            b.record()
            torch.cuda.synchronize()
            if rep:
                best[i] = min(best[i], a.elapsed_time(b))
    for ctx in ctxs:
        pk.proxykv_destroy(ctx)
    assert best[1] < 1.2 * best[0], best


def test_mapper_context_reuse_across_lengths():
    """One context called with a short, a longer and again a shorter sequence (the workspace of every lane grows in
    between; three distinct proxy layers run side by side): same bits as a fresh context each time, and the oracle's
    values on the last one."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="reuse", L_s=3, H_kv=2, H_q=2, L_l=3, H_l=4, N=700, N_q=64, chunk=64,
                             n_planted=0)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(23)
    ctx = _ctx(case, w)
    for N in (700, 2300, 300):
        X = (torch.rand(case.L_s, case.H_kv, N, generator=g) ** 8).to(torch.float32)
        y = pk.proxykv_map(ctx, X.cuda())
        fresh = _ctx(case, w)
        y_fresh = pk.proxykv_map(fresh, X.cuda())
        torch.cuda.synchronize()
        assert torch.equal(y, y_fresh), N
        pk.proxykv_destroy(fresh)
    assert_close(y, oracle.mapper(X, w, case.L_l), "map after reuse, N=300")
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("L,longest,N", [(16, 11500, 4608), (5, 9000, 2049), (33, 700, 100)])
def test_mapper_in_the_workspace_of_a_longer_call(L, longest, N):
    """A shorter call runs in what a longer one has allocated, with as many layers at a time as that holds (16 layers of 4608
    tokens behind one of 11 500: two or three, a fresh context takes eight): same bits as in a fresh context."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="longer", L_s=L, H_kv=2, H_q=2, L_l=L, H_l=4, N=N, N_q=1, chunk=1, n_planted=0)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    g = torch.Generator().manual_seed(500 + N)
    long = (torch.rand(L, case.H_kv, longest, generator=g) ** 8).cuda()
    X = long[:, :, 3:N + 3].contiguous()
    used, fresh = _ctx(case, w), _ctx(case, w)
    pk.proxykv_map(used, long)
    y, y_fresh = pk.proxykv_map(used, X), pk.proxykv_map(fresh, X)
    torch.cuda.synchronize()
    assert torch.equal(y, y_fresh)
    pk.proxykv_destroy(used)
    pk.proxykv_destroy(fresh)


# ----------------------------------------------------------------------------------------------
# whole path
# ----------------------------------------------------------------------------------------------

@pytest.mark.parametrize("L,N", [(2, 700), (16, 300), (1, 3100), (3, 2500)])
def test_mapper_after_scores_that_are_not_finite(L, N):
    """What a longer call with NaN scores leaves in the workspace, behind a shorter call's last rows, does not reach that call's
    results, nor do the NaN scores of one proxy layer reach another layer: small tiles, large tiles, one window and several, the
    last of them cut inside a 64-key tile."""
    g = torch.Generator().manual_seed(N)
    cfg = pk.make_config(L, 4, 2, 64, L, 2, 64)
    w = synth.make_mapper_weights(2, 2)
    x = torch.rand(L, 2, N, generator=g).cuda()
    ctx = pk.proxykv_create(cfg)
    pk.proxykv_set_mapper_weights(ctx, w)
    want = pk.proxykv_map(ctx, x)
    assert bool(torch.isfinite(want).all())
    pk.proxykv_destroy(ctx)
    ctx = pk.proxykv_create(cfg)
    pk.proxykv_set_mapper_weights(ctx, w)
    pk.proxykv_map(ctx, torch.full((L, 2, N + 1200), float("nan"), device="cuda"))
    assert torch.equal(pk.proxykv_map(ctx, x), want)
    if L > 1:
        x[0] = float("nan")
        assert torch.equal(pk.proxykv_map(ctx, x)[1:], want[1:])
    pk.proxykv_destroy(ctx)


def _band_check(y_ref: torch.Tensor, idx_gpu: torch.Tensor, K: int):
    """Every token whose oracle score clears the K-th score by more than the tolerance is kept, every
    token that misses it by more than the tolerance is dropped; exact equality when the K-th and
    (K+1)-th oracle scores are further apart than the tolerance."""
    rows, N = y_ref.shape
    exact = 0
    for r in range(rows):
        srt = torch.sort(y_ref[r], descending=True).values
        sK = float(srt[K - 1])
        tau = 2.0 * (ATOL + RTOL * abs(sK))
        kept = torch.zeros(N, dtype=torch.bool)
        kept[idx_gpu[r].long()] = True
        assert int(kept.sum()) == K and bool((idx_gpu[r][1:] > idx_gpu[r][:-1]).all())
        assert bool(kept[y_ref[r] > sK + tau].all()), f"row {r}: a clearly-in token was dropped"
        assert not bool(kept[y_ref[r] < sK - tau].any()), f"row {r}: a clearly-out token was kept"
        if K < N and float(srt[K - 1] - srt[K]) > tau:
            ref_idx = oracle.topk(y_ref[r:r + 1].float(), K)[0]
            assert torch.equal(idx_gpu[r].cpu(), ref_idx)
            exact += 1
    return exact


def test_prune_tiny_case_end_to_end():
    case = synth.CASES["tiny"]
    q, kc, kr = synth.make_proxy_qk(case)
    k_t, v_t = synth.make_target_kv(case)
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    X_ref, Y_ref, idx_ref, K_ref, V_ref = oracle.prune(q, kc, kr, case.chunk, 0.3, w, k_t, v_t)
    ctx = _ctx(case, w)
    x = torch.empty(case.L_s, case.H_kv, case.N, dtype=torch.float32, device="cuda")
    y = torch.empty(case.L_l, case.H_l, case.N, dtype=torch.float32, device="cuda")
    k_out, v_out, idx, K = pk.proxykv_prune(ctx, q.cuda(), kc.cuda(), kr.cuda(), case.chunk, 0.3, k_t.cuda(), v_t.cuda(),
                                            x_out=x, yhat_out=y)
    torch.cuda.synchronize()
    assert K == 153 == idx_ref.shape[-1]
    assert_close(x, X_ref, "prune.x")
    assert_close(y, Y_ref, "prune.yhat")
    _band_check(Y_ref.view(-1, case.N), idx.cpu().view(-1, K), K)
    # given the GPU's own scores, selection and compaction are exact
    idx_same = oracle.topk(y.cpu().view(-1, case.N), K).view(case.L_l, case.H_l, K)
    assert torch.equal(idx.cpu(), idx_same)
    assert torch.equal(k_out.cpu().view(torch.int16), oracle.compact(k_t, idx_same).view(torch.int16))
    assert torch.equal(v_out.cpu().view(torch.int16), oracle.compact(v_t, idx_same).view(torch.int16))
    # a second call on the same context gives the same bits
    k2, v2, idx2, _ = pk.proxykv_prune(ctx, q.cuda(), kc.cuda(), kr.cuda(), case.chunk, 0.3, k_t.cuda(), v_t.cuda())
    torch.cuda.synchronize()
    assert torch.equal(idx2, idx) and torch.equal(k2.view(torch.int16), k_out.view(torch.int16))


def test_prune_with_the_sum_form_equals_its_stages():
    """reduce = SUM through the fused call: same bits as score -> map -> top-k -> compact called one by one."""
    case = synth.scaled_case(synth.CASES["llama_8k"], name="prune_sum", L_s=2, H_q=4, H_kv=2, d=64, L_l=3, H_l=2, N=700, N_q=500,
                             chunk=200, n_planted=4)
    q, kc, kr = synth.make_proxy_qk(case, device="cuda")
    k_t, v_t = synth.make_target_kv(case, device="cuda")
    w = synth.make_mapper_weights(case.H_kv, case.H_l)
    cfg = pk.config_for_case(case)
    cfg.reduce = pk.PROXYKV_REDUCE_SUM
    ctx = pk.proxykv_create(cfg)
    pk.proxykv_set_mapper_weights(ctx, w)
    x = torch.empty(case.L_s, case.H_kv, case.N, dtype=torch.float32, device="cuda")
    y = torch.empty(case.L_l, case.H_l, case.N, dtype=torch.float32, device="cuda")
    k_out, v_out, idx, K = pk.proxykv_prune(ctx, q, kc, kr, case.chunk, 0.25, k_t, v_t, x_out=x, yhat_out=y)
    torch.cuda.synchronize()
    x2 = pk.proxykv_score(ctx, q, kc, kr, case.chunk)
    y2 = pk.proxykv_map(ctx, x2)
    idx2 = pk.proxykv_topk(ctx, y2.view(-1, case.N), K).view(case.L_l, case.H_l, K)
    k2, v2 = pk.proxykv_compact(ctx, k_t, v_t, idx2)
    torch.cuda.synchronize()
    assert K == 175
    assert torch.equal(x, x2) and torch.equal(y, y2) and torch.equal(idx, idx2)
    assert torch.equal(k_out.view(torch.int16), k2.view(torch.int16)) and torch.equal(v_out.view(torch.int16), v2.view(torch.int16))
    assert_close(x, oracle.score(q.double().cpu(), kc.double().cpu(), kr.double().cpu(), case.chunk, reduce="sum"), "prune sum x")
    pk.proxykv_destroy(ctx)


@pytest.mark.parametrize("L,H_q,H_kv,d", [(1, 4, 2, 64), (16, 32, 8, 64), (28, 12, 2, 128)])
def test_reserve_covers_all_shorter_calls(L, H_q, H_kv, d):
    """A workspace reserved for the longest input serves every shorter one without an allocation, although a shorter one may be
    given more workgroups per key block or more proxy layers per batch: the device's free memory stays what it is."""
    g = torch.Generator().manual_seed(L)
    n_max = 5000
    cfg = pk.make_config(L, H_q, H_kv, d, L, 4, 128)
    ctx = pk.proxykv_create(cfg)
    pk.proxykv_set_mapper_weights(ctx, synth.make_mapper_weights(H_kv, 4))
    q = torch.randn(L, H_q, n_max, d, generator=g).bfloat16().cuda()
    k = torch.randn(L, H_kv, n_max, d, generator=g).bfloat16().cuda()
    x = torch.rand(L, H_kv, n_max, generator=g).cuda()
    calls = []
    for n in (200, 700, 1500, 2049, 4097):
        cut = [t[:, :, :n].contiguous() for t in (q, k, x)]
        calls.append((cut, torch.empty(L, H_kv, n, device="cuda"), torch.empty(L, 4, n, device="cuda")))
    pk.proxykv_reserve(ctx, n_max, n_max)
    pk.proxykv_map(ctx, x)  # code objects and streams are loaded
    pk.proxykv_score(ctx, q, k, k, 512)
    pk.proxykv_score_self(ctx, q, k)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    for (qn, kn, xn), out, yhat in calls:
        pk.proxykv_score(ctx, qn, kn, kn, 512, x_out=out)
        pk.proxykv_score_self(ctx, qn, kn, x_out=out)
        pk.proxykv_map(ctx, xn, yhat=yhat)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free, f"{out.shape[2]} tokens"
    pk.proxykv_destroy(ctx)
