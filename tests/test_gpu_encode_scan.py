"""The scan encoder (csrc/encode_topk_scan.hip) at the edges of its tiles, lists and ranges: bit for bit the same as the fast kernel
(the C entry point without scratch, at these sizes) and as the tiled one (calls of few tokens), which the oracle checks element
by element elsewhere, and against the oracle itself."""
import numpy as np
import pytest
import torch  # noqa: F401  before the library, whose HIP runtime is then torch's

from paper_2601_17702_amd import synth
from tests import parity

NF = 16384


def test_stream_scratch_of_a_shorter_or_narrower_call_is_no_larger():
    """A caller sizes the scratch once for its longest chunk; the ragged last one runs with the same."""
    import paper_2601_17702_amd as s3
    for heads in (1, 3, 8, 32, 100, 256):
        need = [s3.sae_encode_topk_stream_workspace(heads, T) for T in (1, 255, 256, 257, 511, 1000, 2048, 4097, 70000)]
        assert need == sorted(need) and need[0] > 0
    for T in (1, 300, 2048):
        need = [s3.sae_encode_topk_stream_workspace(h, T) for h in (1, 2, 8, 9, 31, 64, 256)]
        assert need == sorted(need)


def test_scratch_holds_what_a_call_can_use():
    """Chunks of under 256 tokens never keep candidate lists there: a place in the queue of the second walk (4 bytes) a token, a few
    bytes a head.  Longer ones: lists of 512 workgroups (436 MB at k = 128) and no more than 4 bytes a token beside them."""
    import paper_2601_17702_amd as s3
    lists = 512 * 512 * 208 * 8
    for heads, T in ((1, 1), (8, 4), (256, 1), (256, 255)):
        assert s3.sae_encode_topk_stream_workspace(heads, T) <= 4 * heads * T + 28 * heads + 5 * 256
    for heads, T in ((256, 2048), (256, 32768), (112, 2048)):
        assert s3.sae_encode_topk_stream_workspace(heads, T) <= lists + 512 * 512 * 4 + 4 * heads * T + (1 << 18)
    for k, cap in ((32, 112), (64, 168), (128, 208)):                # a call without a stream: its own k's lists
        assert 0 < s3.lib().s3_sae_encode_topk_workspace(0, 2048, 128, 16384, k, 256) <= 512 * 512 * (8 * cap + 4) + 4 * 256 * 2048 + (1 << 18)


def plain_without_scratch(x, W, b, k):
    """s3_sae_encode_topk: no scratch, so never the scan encoder but, at this file's sizes, the fast one."""
    import torch
    import paper_2601_17702_amd as s3
    H, T, d = x.shape
    ids = torch.full((H, T, k), -7, dtype=torch.int32, device="cuda")
    vals = torch.full((H, T, k), -7.0, device="cuda")
    rc = s3.lib().s3_sae_encode_topk(s3._ptr(x), 0, T, d, s3._ptr(W), s3._ptr(b), W.shape[1], k, H, s3._ptr(ids), s3._ptr(vals), s3._stream())
    assert rc == 0
    return ids, vals


def problem(H, T, nf, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn(H, nf, 128, generator=g, device="cuda")
    W = (W / W.norm(dim=2, keepdim=True)).to(torch.bfloat16)
    x = torch.randn(H, T, 128, generator=g, device="cuda").to(torch.bfloat16)
    return x, W, 0.01 * torch.randn(H, nf, generator=g, device="cuda")


def plain_takes_the_scan_encoder(H, T, nf, k):
    """By its scratch: the ranges of a call that runs tiled take at most 2^22 entries of 8 bytes."""
    import paper_2601_17702_amd as s3
    return s3.lib().s3_sae_encode_topk_workspace(0, T, 128, nf, k, H) > (8 << 22)


def same(a, b):
    import torch
    torch.cuda.synchronize()
    ok = torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert ok


@pytest.mark.gpu
@pytest.mark.parametrize("H,T,nf,k,plain", [          # plain: a call without a stream takes the scan encoder too
    (1, 256, NF, 1, False),          # one tile, sixteen ranges, the smallest k
    (1, 257, NF, 32, False),         # a tile with one token
    (3, 300, NF, 33, False),         # rows that no 16-byte store can take
    (2, 321, 12288, 64, False),      # ranges that do not divide the stages
    (5, 511, NF, 65, False),
    (9, 449, NF, 128, False),        # heads beyond a multiple of eight, a wavefront with one token
    (16, 256, NF, 32, True),         # as few tokens as a plain call may have
    (9, 456, 8192, 128, True),
    (65, 256, NF, 40, True),         # seven ranges
    (129, 256, NF, 40, True),        # more tiles than are split, one tile a head
    (130, 700, NF, 30, False),       # fewer whole tiles than run at once
    (172, 513, NF, 30, True),        # 516 tiles: a workgroup takes a second one; one build each
    (172, 513, NF, 48, True),
    (172, 513, NF, 100, True),
    (130, 900, 12288, 64, True),     # 520 tiles, four a head: the second turn is moved on by one
])
@pytest.mark.timeout(100)
def test_streamed_and_plain_calls_equal_the_other_kernels(H, T, nf, k, plain):
    import paper_2601_17702_amd as s3
    x, W, b = problem(H, T, nf, H * 1000 + T + k)
    want = plain_without_scratch(x, W, b, k)
    if H < 10:
        same(tiled_rows(x, W, b, k), want)
    assert plain_takes_the_scan_encoder(H, T, nf, k) == plain
    same(s3.sae_encode_topk(x, W, b, k), want)
    hint = s3.new_tau_hint(H)
    for _ in range(3):                       # without a bound, then with one as tight as it gets
        same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)
        h = hint.cpu().numpy()
        assert np.all(np.isfinite(h).sum(axis=1) == 1)
        # the carried value is a lower bound of the k-th values
        kth = want[1][:, :, -1].cpu().numpy()
        assert np.all(np.where(np.isfinite(h[:, 1]), h[:, 1], -np.inf) <= kth.min(axis=1) + 1e-6)


@pytest.mark.gpu
@pytest.mark.parametrize("H,T,nf,k", [
    (128, 256, 12544, 48),           # 512 groups of 64 tokens: the most whose samples four wavefronts share
    (103, 300, 12544, 48),           # 515: four groups a workgroup, 49 sampled stages, three wavefronts without a token
    (103, 300, 12544, 100),
    (130, 300, 16640, 30),           # 65 sampled stages
    (1, 33000, 12544, 64),           # one head
])
@pytest.mark.timeout(100)
def test_first_thresholds_from_odd_samples(H, T, nf, k):
    """Stages sampled in pairs, the last without a partner; biases at an odd float; results exact, also from call to call."""
    import torch
    import paper_2601_17702_amd as s3
    x, W, b = problem(H, T, nf, H + T + k)
    b = torch.cat([torch.zeros(1, device="cuda"), b.reshape(-1)])[1:].view(H, nf)
    want = plain_without_scratch(x, W, b, k)
    hint = s3.new_tau_hint(H)
    same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)
    hint.fill_(float("-inf"))
    same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)


@pytest.mark.gpu
@pytest.mark.parametrize("H,T,k", [(8, 512, 32), (70, 512, 48), (70, 512, 128)])
@pytest.mark.timeout(100)
def test_some_tokens_start_too_high(H, T, k):
    """A bound in the middle of the tokens' thresholds: some wavefronts of a workgroup have tokens to walk again, some have none."""
    import torch
    import paper_2601_17702_amd as s3
    x, W, b = problem(H, T, NF, 5 + k)
    want = plain_without_scratch(x, W, b, k)
    r = want[1][:, :, -1] / x.float().norm(dim=2)
    for q in (0.002, 0.3, 0.99):
        hint = s3.new_tau_hint(H)
        hint[:, 0] = torch.quantile(r, q, dim=1) / 0.96          # the call starts 4 % below it
        same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)
    for bad in (float("inf"), float("nan"), -1e30):
        hint = torch.full((H, 2), bad, device="cuda")
        same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)


@pytest.mark.gpu
@pytest.mark.parametrize("H,T,k,plain", [
    (2, 300, 32, False),
    (16, 257, 32, True),             # ranges and their join
    (172, 520, 32, True),            # whole tiles
    (70, 256, 64, True),             # seven ranges
    (66, 300, 128, True),            # whole tiles
])
@pytest.mark.timeout(100)
def test_ties_masked_features_and_sorted_dictionaries(H, T, k, plain):
    import torch
    import paper_2601_17702_amd as s3
    assert plain_takes_the_scan_encoder(H, T, NF, k) == plain
    x, W, b = problem(H, T, NF, 77 + k)

    def check(x, W, b, want):                # with a sample's thresholds, and with a stream's
        same(s3.sae_encode_topk(x, W, b, k), want)
        hint = s3.new_tau_hint(H)
        for _ in range(2):
            same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)

    # every pre-activation the same: the lowest ids, from lists that are cut again and again
    zero = torch.zeros_like(W)
    check(x, zero, torch.ones_like(b), plain_without_scratch(x, zero, torch.ones_like(b), k))
    del zero
    # few different values
    g = torch.Generator(device="cuda").manual_seed(3)
    xi = torch.randint(-1, 2, x.shape, generator=g, device="cuda").to(torch.bfloat16)
    Wi = W[:, :64].sign().repeat(1, NF // 64, 1).contiguous()
    check(xi, Wi, torch.zeros_like(b), plain_without_scratch(xi, Wi, torch.zeros_like(b), k))
    del Wi
    # ascending and descending biases: all that counts comes last, or first (the sample's thresholds are then far off)
    for sign in (1.0, -1.0):
        bs = (sign * torch.linspace(-9, 9, NF, device="cuda")).repeat(H, 1).contiguous()
        check(x, W, bs, plain_without_scratch(x, W, bs, k))
    # features masked with -inf: first all but a hundred, then all but fewer than k: rows are filled with the lowest other ids
    for left in (200, k - 5):
        bm = torch.full_like(b, float("-inf"))
        bm[:, torch.randperm(NF, generator=torch.Generator().manual_seed(1))[:left].cuda()] = 0.0
        check(x, W, bm, tiled_rows(x, W, bm, k))


@pytest.mark.gpu
@pytest.mark.parametrize("H,T,k", [(16, 300, 32), (172, 520, 32), (70, 256, 64), (66, 300, 128)])
@pytest.mark.timeout(100)
def test_tokens_of_nan_and_overflowing_ones(H, T, k):
    """A token of NaN has no element, one whose products overflow has elements of +inf and NaN beside finite ones; the rows of the
    other tokens of their tiles and the bounds carried on are not touched by them."""
    import torch
    import paper_2601_17702_amd as s3
    x, W, b = problem(H, T, NF, 5 + T)
    clean = s3.new_tau_hint(H)
    s3.sae_encode_topk_stream(x, W, b, k, clean)
    x[:, 3, 17] = float("nan")
    x[0, T - 1, 0] = float("inf")
    x[:, 130] = 2e38 * x[:, 130].sign()
    want = tiled_rows(x, W, b, k)
    same(s3.sae_encode_topk(x, W, b, k), want)
    hint = s3.new_tau_hint(H)
    for _ in range(2):
        same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)
        assert not torch.any(torch.isnan(hint)) and torch.all(torch.isfinite(hint).sum(dim=1) == 1)
        assert torch.all(hint[:, 0] <= 1.001 * clean[:, 0] + 1.0)


@pytest.mark.gpu
@pytest.mark.parametrize("H,T,k", [(12, 300, 32), (70, 520, 64), (70, 520, 128), (140, 520, 32)])
@pytest.mark.timeout(100)
def test_heads_with_and_without_a_bound_and_outputs_at_any_int(H, T, k):
    """Half of the heads start from a carried bound, the others from the sample; rows of a multiple of four that are not aligned to 16
    bytes; and scratch that calls of other shapes have used before on the same stream."""
    import torch
    import paper_2601_17702_amd as s3
    x, W, b = problem(H, T, NF, 3 * k + T)
    want = plain_without_scratch(x, W, b, k)
    hint = s3.new_tau_hint(H)
    s3.sae_encode_topk_stream(x, W, b, k, hint)
    full = hint.clone()
    ws = torch.randint(0, 256, (s3.sae_encode_topk_stream_workspace(H, T),), dtype=torch.uint8, device="cuda")
    ids = torch.full((H * T * k + 8,), -7, dtype=torch.int32, device="cuda")
    vals = torch.full((H * T * k + 8,), -7.0, device="cuda")
    for off in (0, 1, 2):
        hint = full.clone()
        hint[1::2] = float("-inf")
        o = (ids[off:off + H * T * k].view(H, T, k), vals[off:off + H * T * k].view(H, T, k))
        same(s3.sae_encode_topk_stream(x, W, b, k, hint, ws, *o), want)
        assert torch.all(torch.isfinite(hint).sum(dim=1) == 1)
        assert torch.all(ids[off + H * T * k:] == -7) and torch.all(vals[off + H * T * k:] == -7)
        ids.fill_(-7), vals.fill_(-7)
        s3.sae_encode_topk_stream(x[:3, :257].contiguous(), W[:3], b[:3], 7, s3.new_tau_hint(3), ws)     # other lists in the same place


@pytest.mark.gpu
@pytest.mark.parametrize("H,T,k", [(8, 512, 32), (70, 300, 48), (66, 600, 128), (130, 520, 20)])
@pytest.mark.timeout(100)
def test_rows_of_zeros_and_outliers_without_biases(H, T, k):
    """A row of zeros has all pre-activations equal: it starts too high wherever the others' thresholds are, and its lists are full of
    ties inside the walk.  Rows that are a multiple of the others meet a bound that is far too low and fill theirs over and over."""
    import torch
    import paper_2601_17702_amd as s3
    x, W, b = problem(H, T, NF, 31 + k)
    b.zero_()
    x[:, 3] = 0
    x[:, T - 1] = 0
    x[:, 17::64] *= 40
    want = plain_without_scratch(x, W, b, k)
    assert torch.all(want[0][:, T - 1] == torch.arange(k, device="cuda", dtype=torch.int32))
    hint = s3.new_tau_hint(H)
    for _ in range(2):
        same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)
    hint.fill_(float("-inf"))
    hint[:, 1] = 1.0                         # a bound on the threshold itself: outliers bring half of all features
    same(s3.sae_encode_topk_stream(x, W, b, k, hint), want)


def tiled_rows(x, W, b, k):
    """The tiled kernel by a call of few tokens at a time (64 rows of every head)."""
    import torch
    import paper_2601_17702_amd as s3
    out = [s3.sae_encode_topk(x[h:h + 1, t:t + 64].contiguous(), W[h:h + 1], b[h:h + 1], k) for h in range(x.shape[0]) for t in range(0, x.shape[1], 64)]
    per = (x.shape[1] + 63) // 64
    rows = [torch.cat([o[i] for o in out[h * per:(h + 1) * per]], dim=1) for i in (0, 1) for h in range(x.shape[0])]
    return torch.cat(rows[:x.shape[0]]), torch.cat(rows[x.shape[0]:])


@pytest.mark.gpu
@pytest.mark.parametrize("name,T,k", [("c2_llama8b", 1030, 32), ("c3_long", 1000, 32), ("c6_paper_sae", 520, 128)])
@pytest.mark.timeout(100)
def test_against_the_oracle(name, T, k):
    import torch
    import paper_2601_17702_amd as s3
    w = synth.shrink(synth.WORKLOADS[name], T=T, L=2 * T, n_feat=NF)
    heads = [0, 1, 5, 7]
    W, b = np.stack([synth.gen_w_enc(w, h) for h in heads]), np.stack([synth.gen_b_enc(w, h) for h in heads])
    Wg, bg, hint = parity.to_gpu(W, w.dtype), parity.to_gpu(b, "fp32"), s3.new_tau_hint(len(heads))
    rows = np.r_[0:40, T - 40:T]             # the oracle's own time: some rows of each chunk
    for c in range(2):
        x = np.stack([synth.gen_keys(w, h, c) for h in heads])
        ids, vals = s3.sae_encode_topk_stream(parity.to_gpu(x, w.dtype), Wg, bg, k, hint)
        torch.cuda.synchronize()
        parity.check_encode(ids.cpu().numpy()[:, rows], vals.cpu().numpy()[:, rows], x[:, rows], W, b, k, w.dtype)
