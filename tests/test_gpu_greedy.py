"""Scoring and peaks around the sizes at which another way is taken.  The greedy searches that bring the blocks their choices can
lie in into LDS: numbers of blocks and of slots around the sizes at which another build or another kernel takes over, more equal
block maxima than there are slots, choices that end among equal values.  The gather: few and many query pairs, lists in parts,
segments around the numbers of vectors and of lists that are taken together, very long lists, many heads.  The pooling over the
groups.  And times of calls that differ in one of these alone."""
import numpy as np
import pytest

from oracle import s3_oracle as orc
from tests.test_gpu_index_score import check_score, gpu_index, oracle_score, run_gpu_score
from tests.test_gpu_select import oracle_select

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,span_len,top_b,nms", [
    (2 * 64 + 31, 32, 4, True),              # three blocks, all in slots
    (64 * 64 + 7, 8, 65, False),             # 65 slots asked for of 64 blocks
    (128 * 64 + 65, 66, 43, True),           # 127 of 128 blocks: two slots per lane
    (20_000, 64, 86, True),                  # 256 of 312 blocks, the most that LDS holds
    (20_000, 64, 87, True),                  # 259: maxima in registers, windows in memory
    (20_000, 300, 60, True),
    (16_384, 64, 4, True), (16_384, 64, 5, True),      # from so many spans on in LDS
    (16_384, 501, 10, True), (16_384, 501, 11, True), (9000, 768, 40, True), (16_384, 900, 30, True), (16_384, 901, 30, True),      # the longer, the more
    (65_536 + 63, 64, 16, True),             # 1024 maxima, one per thread; one more below
    (65_536 + 64, 64, 16, True),
    ((1 << 18) + 63, 64, 40, True),          # four per thread; sixteen below
    ((1 << 18) + 64, 64, 80, True),
    ((1 << 20) + 63, 64, 30, True),          # the most maxima
])
def test_spans_around_the_numbers_of_slots(T, span_len, top_b, nms):
    rng = np.random.default_rng(T + top_b)
    n = min(T, 20_000)
    at = np.sort(rng.permutation(T)[:n])
    ids = np.zeros((1, T, 1), np.int32)
    ids[0, at, 0] = 1 + rng.permutation(n)
    qids = (1 + np.arange(n, dtype=np.int32))[None, :, None].copy()
    qvals = (rng.random((1, n, 1)) + 0.01).astype(np.float32)
    ix = gpu_index(ids, n + 1)
    S, W, st_o, sc_o = oracle_score(ids, qids, qvals, n + 1, T, span_len, top_b, 0, nms)
    out = run_gpu_score(ix, qids, qvals, T, span_len, top_b, 0, nms)
    check_score(out, S, W, st_o, sc_o, span_len, nms)
    assert out[0][:out[2]].tolist() == list(st_o)


@pytest.mark.parametrize("T,span_len,top_b", [(20_000, 40, 12), (70_000, 64, 30)])
def test_equal_spans_are_taken_from_the_front(T, span_len, top_b):
    """One feature in every position: all windows are equal, and there are more equal block maxima than slots."""
    ids = np.zeros((1, T, 1), np.int32)
    ix = gpu_index(ids, 2)
    st, _, nf, _ = run_gpu_score(ix, np.zeros((1, 1, 1), np.int32), np.ones((1, 1, 1), np.float32), T, span_len, top_b, 0, True)
    assert nf == top_b and st.tolist() == [i * span_len for i in range(top_b)]


def plateaus(rng, n, high):
    """0 / 1 in long stretches, with `high` positions above: most choices fall among equal values."""
    v = np.zeros(n, np.int32)
    edge = np.sort(rng.choice(n, 12, replace=False))
    for lo, hi in zip(edge[::2], edge[1::2]):
        v[lo:hi] = 1
    v[rng.choice(n, high, replace=False)] = 2 + np.arange(high)
    return v


@pytest.mark.parametrize("T,span_len,top_b,high", [
    (20_000, 9, 20, 3), (20_000, 9, 20, 0),  # 64 slots
    (20_000, 9, 60, 7),                      # 128
    (20_000, 34, 80, 30), (300, 34, 80, 1),  # 256; more asked for than there are
    (70_000, 34, 80, 5),                     # four maxima per thread
])
def test_spans_that_end_among_equal_ones(T, span_len, top_b, high):
    """Fewer windows stand out than are asked for: the others come in ascending order."""
    ids = plateaus(np.random.default_rng(T + top_b + high), T, high).reshape(1, T, 1)
    n_feat = high + 3
    qids = np.arange(1, n_feat, dtype=np.int32).reshape(1, -1, 1).copy()
    qvals = np.linspace(1.0, 3.0, qids.size).astype(np.float32).reshape(qids.shape)
    ix = gpu_index(ids, n_feat)
    S, W, st_o, sc_o = oracle_score(ids, qids, qvals, n_feat, T, span_len, top_b, 0, True)
    out = run_gpu_score(ix, qids, qvals, T, span_len, top_b, 0, True)
    check_score(out, S, W, st_o, sc_o, span_len, True)
    # a position has one weight: as whole numbers of 40 bits the window sums are exact in fp64, and equal where members are
    fixed = np.concatenate([[0], np.cumsum(np.rint(S / S.max() * 2.0 ** 40))])
    st_x, _ = orc.topb(fixed[span_len:] - fixed[:-span_len], span_len, top_b)
    assert out[0][:out[2]].tolist() == st_x.tolist()


@pytest.mark.parametrize("L,radius,n_centers,high", [
    (20_000, 8, 20, 3), (20_000, 8, 20, 0),  # 64 slots
    (20_000, 8, 60, 7),                      # 128
    (20_000, 33, 60, 30), (70_000, 33, 60, 5),      # 256
    (70_000, 33, 150, 40), (70_000, 40, 150, 0),    # 512
])
def test_peaks_that_end_among_equal_ones(L, radius, n_centers, high):
    check_peaks(plateaus(np.random.default_rng(L + n_centers + high), L, high).astype(np.float32), radius, n_centers)


@pytest.mark.parametrize("L,radius,n_centers", [
    (40_000, 271, 8), (40_000, 271, 9), (40_000, 272, 9), (40_000, 272, 10),      # from so many centres on in LDS
    (90_000, 500, 16), (90_000, 500, 17), (32_768, 1000, 40),
    (45_000, 64, 171), (45_000, 300, 52), (40_000, 300, 49),     # 511 of 704 blocks asked for; 562, few centres; 529 of 625
    (36_864, 300, 52),                       # 562 of 576
    (300_000, 130, 40),                      # five maxima per thread
])
def test_peaks_around_the_radii(L, radius, n_centers):
    check_peaks(np.random.default_rng(L + radius).random(L).astype(np.float32) ** 2, radius, n_centers)


def best_us(fn, reps=5, calls=10):
    import torch
    fn()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1000 / calls)
    return best


@pytest.mark.parametrize("span_len,top_b", [(16, 64), (32, 8), (64, 64)])
def test_a_query_without_matches_costs_what_another_one_does(span_len, top_b):
    """All windows are equal: half a microsecond a choice, and at most twice that here."""
    import torch
    T = 16_384
    ids = (np.arange(T, dtype=np.int32) * 7 % 4096).reshape(1, T, 1)
    ix = gpu_index(ids, 4096)
    qids = torch.arange(512, dtype=torch.int32, device="cuda").view(1, 512, 1)
    some, none = torch.rand(1, 512, 1, device="cuda"), torch.zeros(1, 512, 1, device="cuda")
    us = [best_us(lambda: ix.coactivate_score(qids, q, T, span_len, top_b)) for q in (some, none)]
    assert us[1] < us[0] + 1.2 * top_b + 5, us


def look_up(H, L, nq, span_len, k=16, n_feat=8192):
    """A look-up of four spans, to be timed: features evenly drawn, lists of L k / n_feat positions."""
    import torch
    import paper_2601_17702_amd as s3
    ix = s3.Index(H, n_feat, k, L)
    for t in range(0, L, 32_768):
        start = torch.randint(0, n_feat, (H, min(32_768, L - t), 1), device="cuda", dtype=torch.int32)
        ix.append(((start + n_feat // k * torch.arange(k, device="cuda", dtype=torch.int32)) % n_feat).contiguous(), base_pos=t)
    ix.finalize()
    q = torch.randint(0, n_feat, (H, nq, k), device="cuda", dtype=torch.int32)
    v = torch.rand(H, nq, k, device="cuda")
    ws = torch.empty(ix.score_workspace(L), dtype=torch.uint8, device="cuda")
    return best_us(lambda: ix.coactivate_score(q, v, L, span_len, 4, want_scores=True, ws=ws))


@pytest.mark.parametrize("a,b,factor", [
    ((64, 16_384, 16, 1024), (64, 16_384, 16, 64), 1.5),       # longer windows are pooled by as many workgroups
    ((256, 8000, 16, 4000), (256, 8000, 16, 64), 1.5),
    ((1, 1_000_000, 2, 64), (1, 250_000, 2, 64), 1.6),         # tiles grow with the context
    ((64, 16_384, 16, 64), (64, 16_384, 2, 64), 1.3),         # lists are shared where that is worth a further array
], ids=str)
def test_times_of_look_ups(a, b, factor):
    """(heads, positions, queries, window) and one that takes nearly as long."""
    us = look_up(*b), look_up(*a), look_up(*b), look_up(*a)
    us = min(us[1], us[3]), min(us[0], us[2])
    assert us[0] < factor * us[1], us


@pytest.mark.parametrize("kind", ["none", "dropped", "one"])
def test_queries_that_name_little_share_no_lists(kind):
    """179 queries whose lists are all empty of weight, too long, or but one, in 13 heads: as fast as two of them."""
    import torch
    H, L, k, n_feat = 13, 28_741, 32, 1203
    rng = np.random.default_rng(0)
    ids = ((rng.integers(0, n_feat, (H, L, 1)) + np.arange(k) * (n_feat // k)) % n_feat).astype(np.int32)
    ix = gpu_index(ids, n_feat)
    us, S = [], []
    for nq in (2, 179):
        qids = torch.from_numpy(np.random.default_rng(1).integers(0, n_feat, (H, 179, k)).astype(np.int32)).cuda()[:, :nq].contiguous()
        qvals = torch.zeros(H, nq, k, device="cuda")
        if kind == "dropped":
            qvals[:] = 1
        if kind == "one":
            qvals[7, 1, 3] = 1
        ws = torch.empty(ix.score_workspace(L), dtype=torch.uint8, device="cuda")
        call = lambda: ix.coactivate_score(qids, qvals, L, 300, 4, max_freq=50 if kind == "dropped" else 0, want_scores=True, ws=ws)
        S.append(call()[3])
        us.append(best_us(call))
    assert torch.equal(S[0], S[1]) and (float(S[0].max()) > 0) == (kind == "one")
    assert us[1] < 1.25 * us[0] + 4, us


@pytest.mark.parametrize("radius,n_centers", [(8, 9), (8, 40), (48, 128), (64, 40)])
def test_a_level_curve_costs_what_another_one_does(radius, n_centers):
    import torch
    import paper_2601_17702_amd as s3
    g = s3.smoothing_kernel(s3.KERNEL_BOX, 1)
    us = [best_us(lambda: s3.select_spans(S, g, n_centers, radius, 0.5, 64)) for S in (torch.rand(32_768, device="cuda"), torch.ones(32_768, device="cuda"))]
    assert us[1] < us[0] + 1.2 * n_centers + 5, us


@pytest.mark.parametrize("L,radius", [(70_000, 2000), (300_000, 2000), (70_000, 1000)])
def test_one_more_centre_of_a_large_radius(L, radius):
    import torch
    import paper_2601_17702_amd as s3
    g, S = s3.smoothing_kernel(s3.KERNEL_GAUSSIAN, 48), torch.rand(L, device="cuda")
    us = [best_us(lambda: s3.select_spans(S, g, n, radius, 0.5, 64)) for n in (8, 9)]
    assert us[1] < 1.2 * us[0] + 2, us


@pytest.mark.parametrize("L,radius,n_centers,levels", [
    (36_864, 64, 40, 3), (36_865, 64, 40, 3),      # 576 blocks, all in slots; one more
    (40_000, 64, 192, 2), (40_000, 64, 193, 2),    # 574 and 577 slots asked for
    (50_000, 33, 22, 0),                           # 64 slots, all densities equal
    (65_536, 1, 100, 2), (65_537, 1, 100, 2),      # 1024 maxima, one per thread; one more
    (70_000, 0, 64, 1), (70_000, 0, 65, 1),        # no suppression beyond the centre: 64 and 65 slots
    (1 << 20, 64, 130, 4), ((1 << 20) + 1, 64, 130, 4),      # sixteen per thread; tiles of two blocks
])
def test_peaks_around_the_numbers_of_slots(L, radius, n_centers, levels):
    """Few distinct densities, so that block maxima tie; `levels` 0: one."""
    rng = np.random.default_rng(L + n_centers)
    check_peaks(rng.integers(0, levels + 1, L).astype(np.float32) if levels else np.ones(L, np.float32), radius, n_centers)


def check_peaks(S, radius, n_centers):
    import torch
    import paper_2601_17702_amd as s3
    g = s3.smoothing_kernel(s3.KERNEL_BOX, 1)
    c, dc, lo, hi, nf, D = s3.select_spans(torch.from_numpy(S).cuda(), g, n_centers, radius, 0.5, 70, want_density=True)
    torch.cuda.synchronize()
    D32, c_o, pk_o, lo_o, hi_o = oracle_select(S, g.cpu().numpy(), n_centers, radius, 0.5, 70)
    n = int(nf.item())
    assert np.array_equal(D.cpu().numpy(), D32) and n == len(c_o)
    assert np.array_equal(c.cpu().numpy()[:n], c_o) and np.array_equal(dc.cpu().numpy()[:n], pk_o.astype(np.float32))
    assert np.array_equal(lo.cpu().numpy()[:n], lo_o) and np.array_equal(hi.cpu().numpy()[:n], hi_o)


@pytest.mark.parametrize("H,T,span_len", [
    (2, 5000, 64), (5, 3000, 700), (9, 2500, 100), (17, 4100, 33), (25, 1000, 10),       # arrays in batches of sixteen and four
    (24, 1300, 682), (24, 1300, 683), (100, 900, 163), (100, 900, 164),      # summed by the pooling, and before it
    (1, 40_000, 128), (1, 70_000, 2000), (1, 300_000, 64), (1, 9000, 4096), (3, 9000, 4097),      # tiles of 256 to 2048 windows
])
def test_pooling_over_the_groups(H, T, span_len):
    rng = np.random.default_rng(H * T + span_len)
    ids = ((rng.integers(0, 25, (H, T, 1)) + np.arange(2) * 25) % 50).astype(np.int32)
    qids = rng.integers(0, 50, (H, 3, 2)).astype(np.int32)
    qvals = rng.random((H, 3, 2)).astype(np.float32)
    ix = gpu_index(ids, 50)
    S, W, st_o, sc_o = oracle_score(ids, qids, qvals, 50, T, span_len, 8, 0, True)
    check_score(run_gpu_score(ix, qids, qvals, T, span_len, 8, 0, True), S, W, st_o, sc_o, span_len, True)


@pytest.mark.parametrize("H,T,k,n_feat,nq,hot", [
    (1, 3000, 32, 256, 32, 0),           # 1024 query pairs, the most for a thread each; a head's lists in parts
    (2, 3000, 25, 300, 41, 0),           # 1025
    (1, 40_000, 16, 4096, 9, 8),         # lists that fill whole position blocks, beside short ones
    (1, 20_000, 100, 400, 20, 100),      # a hundred of them
    (3, 700, 7, 17_000, 64, 0),          # two feature ranges
])
def test_gather_of_short_and_long_lists(H, T, k, n_feat, nq, hot):
    """Segments of every alignment and length, plain and compact; `hot` features are in every token."""
    rng = np.random.default_rng(T + k)
    ids = np.empty((H, T, k), np.int32)
    for h in range(H):
        if hot >= k - 1:
            ids[h] = np.arange(k, dtype=np.int32)[None, :]
        elif hot:
            ids[h, :, :hot] = np.arange(hot)
            start = rng.integers(0, n_feat - hot, T)
            ids[h, :, hot:] = hot + (start[:, None] + np.arange(k - hot) * ((n_feat - hot) // (k - hot))) % (n_feat - hot)
        else:
            start = (n_feat * rng.random(T) ** 2).astype(np.int64)
            ids[h] = (start[:, None] + np.arange(k) * (n_feat // k)) % n_feat
    qids = np.stack([np.stack([rng.choice(n_feat, k, replace=False) for _ in range(nq)]) for _ in range(H)]).astype(np.int32)
    if hot:
        qids[:, 0, :] = np.arange(k)
    qvals = np.maximum(rng.random((H, nq, k)) - 0.1, 0).astype(np.float32)
    ix = gpu_index(ids, n_feat, chunks=[7000] * (T // 7000 + 1))
    S, W, st_o, sc_o = oracle_score(ids, qids, qvals, n_feat, T, 40, 12, 0, True)
    plain = run_gpu_score(ix, qids, qvals, T, 40, 12, 0, True)
    check_score(plain, S, W, st_o, sc_o, 40, True)
    if T > 16384:                                              # the compact form needs two position blocks
        cx = ix.compact(0)
        whole = run_gpu_score(cx, qids, qvals, T, 40, 12, 0, True)
        short = run_gpu_score(cx, qids, qvals, T - 130, 40, 12, 0, True)      # the last positions are cut off
        assert np.array_equal(whole[3], plain[3]) and np.array_equal(whole[0], plain[0])
        assert np.array_equal(short[3], plain[3][:T - 130])


@pytest.mark.parametrize("n_lists", [1024, 1025])
def test_gather_of_as_many_lists_as_are_numbered_together(n_lists):
    """One head, one part: 1024 segments at a time."""
    rng = np.random.default_rng(n_lists)
    T, n_feat = 1500, 1100
    ids = np.concatenate([np.arange(n_feat), rng.integers(0, n_feat, T - n_feat)]).astype(np.int32)
    ids = rng.permutation(ids).reshape(1, T, 1)
    qids = rng.permutation(n_feat)[:n_lists].astype(np.int32).reshape(1, -1, 1).copy()
    qvals = (rng.random(qids.shape) + 0.1).astype(np.float32)
    S, W, st_o, sc_o = oracle_score(ids, qids, qvals, n_feat, T, 16, 8, 0, True)
    check_score(run_gpu_score(gpu_index(ids, n_feat), qids, qvals, T, 16, 8, 0, True), S, W, st_o, sc_o, 16, True)


def test_gather_of_segments_around_a_wavefronts_load():
    """A wavefront has 256 vectors of four postings in flight: lists of 1023 to 1025 postings at each alignment, and longer ones,
    each with a weight of its own.  One position block, one part."""
    rng = np.random.default_rng(3)
    lengths = [1023, 1, 1024, 2, 1025, 3, 1024, 1, 1023, 4, 1022, 1, 1026, 2, 1021, 1, 3000, 1, 2048]
    T, n_feat = sum(lengths), 16 * len(lengths)
    ids = rng.permutation(np.repeat(np.arange(len(lengths)), lengths)).astype(np.int32).reshape(1, T, 1)
    qids = np.arange(len(lengths), dtype=np.int32).reshape(1, -1, 1).copy()
    qvals = (1 + rng.random(qids.shape)).astype(np.float32)
    S, W, st_o, sc_o = oracle_score(ids, qids, qvals, n_feat, T, 16, 8, 0, True)
    check_score(run_gpu_score(gpu_index(ids, n_feat), qids, qvals, T, 16, 8, 0, True), S, W, st_o, sc_o, 16, True)


def test_gather_of_whole_lists_of_many_tokens():
    """More than 2^20 tokens at given positions: no block table, and the lists of one head at a time."""
    rng = np.random.default_rng(8)
    T, n_feat, H = (1 << 20) + 300, 16, 2
    ids = rng.integers(0, n_feat, (H, T, 1)).astype(np.int32)
    qids = np.stack([rng.permutation(n_feat)[:5] for _ in range(H)]).astype(np.int32).reshape(H, 5, 1).copy()
    qvals = (1 + rng.random(qids.shape)).astype(np.float32)
    at = rng.permutation(T).astype(np.int32)
    for positions in (at, np.sort(at)):
        ix = gpu_index(ids, n_feat, positions=positions)
        S, W, st_o, sc_o = oracle_score(ids, qids, qvals, n_feat, T, 64, 8, 0, True, positions=positions)
        full = run_gpu_score(ix, qids, qvals, T, 64, 8, 0, True)
        check_score(full, S, W, st_o, sc_o, 64, True)
        for L in (16_384, 10_001):
            assert np.array_equal(run_gpu_score(ix, qids, qvals, L, 64, 8, 0, True)[3], full[3][:L])


def test_gather_of_more_heads_than_are_looked_at_together():
    """1200 heads of two feature ranges in three groups: 800 pairs a group.  One posting list of every head is queried."""
    import torch
    import paper_2601_17702_amd as s3
    H, T, n_feat, L = 1200, 8, 16_400, 64 * 16384 + 77
    rng = np.random.default_rng(4)
    ids = rng.integers(0, n_feat, (H, T, 1)).astype(np.int32)
    at = np.sort(rng.choice(L, T, replace=False)).astype(np.int32)
    ix = s3.Index(H, n_feat, 1, T)
    ix.append(torch.from_numpy(ids).cuda(), positions=torch.from_numpy(at).cuda())
    ix.finalize()
    slot = rng.integers(0, T, H)
    qids = ids[np.arange(H), slot][:, None, :].copy()
    qvals = rng.integers(1, 1000, (H, 1, 1)).astype(np.float32)
    _, _, _, S = ix.coactivate_score(torch.from_numpy(qids).cuda(), torch.from_numpy(qvals).cuda(), L, 64, 4, want_scores=True)
    torch.cuda.synchronize()
    want = np.zeros(L)
    for h in range(H):
        hit = ids[h, :, 0] == qids[h, 0, 0]
        want[at[hit]] += qvals[h, 0, 0] / (1.0 + np.log(1.0 + hit.sum()))
    assert np.allclose(S.cpu().numpy(), want, rtol=1e-5, atol=1e-30)
