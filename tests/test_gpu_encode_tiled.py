"""The tiled encoder (every shape outside the streamed bf16 / d_head 128 kernel): edges of its 32-token tiles, 256-feature
chunks and feature ranges, against the fp64 oracle, and the split over workgroups against the unsplit call bit for bit."""
import ctypes as C

import numpy as np
import pytest

from paper_2601_17702_amd import synth
from tests import parity

pytestmark = pytest.mark.gpu


def unsplit(s3, x, W, b, k):
    """The call without scratch: one workgroup walks all features of its tokens."""
    import torch
    heads, T, d = x.shape
    ids = torch.full((heads, T, k), -7, dtype=torch.int32, device="cuda")
    vals = torch.full((heads, T, k), -7.0, device="cuda")
    p = lambda t: C.c_void_p(t.data_ptr())
    s3._check(s3.lib().s3_sae_encode_topk(p(x), s3._dtype_code(x), T, d, p(W), p(b), W.shape[1], k, heads, p(ids), p(vals),
                                          s3._stream()))
    return ids, vals


@pytest.mark.parametrize("dtype,d,heads,T,n_feat,k", [
    ("bf16", 128, 3, 1, 257, 64),        # the last range holds one feature, fewer than k
    ("bf16", 128, 1, 33, 20001, 61),     # many ranges, one token in the second tile
    ("bf16", 64, 9, 31, 513, 65),        # lists of 256, heads beyond a multiple of 8
    ("bf16", 256, 2, 64, 2303, 121),     # the largest k at width 256, ragged last chunk
    ("fp32", 64, 2, 32, 4097, 128),
    ("fp32", 128, 1, 95, 1000, 16),
    ("fp32", 256, 5, 7, 1025, 78),
    ("fp32", 256, 1, 700, 300, 1),
])
def test_split_and_unsplit_calls_match_the_oracle(dtype, d, heads, T, n_feat, k):
    import torch
    import paper_2601_17702_amd as s3
    rng = np.random.default_rng(d + n_feat + k + T)
    x = synth.to_storage(rng.standard_normal((heads, T, d)).astype(np.float32), dtype)
    W = synth.to_storage((rng.standard_normal((heads, n_feat, d)) / np.sqrt(d)).astype(np.float32), dtype)
    b = (0.1 * rng.standard_normal((heads, n_feat))).astype(np.float32)
    xg, Wg, bg = parity.to_gpu(x, dtype), parity.to_gpu(W, dtype), parity.to_gpu(b, "fp32")
    ids, vals = s3.sae_encode_topk(xg, Wg, bg, k)
    ids1, vals1 = unsplit(s3, xg, Wg, bg, k)
    torch.cuda.synchronize()
    assert torch.equal(ids, ids1) and torch.equal(vals, vals1)
    parity.check_encode(ids.cpu().numpy(), vals.cpu().numpy(), x, W, b, k, dtype)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 256), ("fp32", 128)])
@pytest.mark.parametrize("k", [5, 64, 78])
def test_ties_across_chunks_and_ranges_take_the_lower_id(dtype, d, k):
    """Few different feature vectors of small integers: exact sums, runs of equal values longer than the lists."""
    import torch
    import paper_2601_17702_amd as s3
    from oracle import s3_oracle as orc
    rng = np.random.default_rng(k + d)
    n_feat, T = 1500, 37
    base = rng.integers(-2, 3, (3, d)).astype(np.float32)
    W = synth.to_storage(base[rng.integers(0, 3, n_feat)][None], dtype)
    x = synth.to_storage(rng.integers(-2, 3, (1, T, d)).astype(np.float32), dtype)
    b = np.zeros((1, n_feat), np.float32)
    xg, Wg, bg = parity.to_gpu(x, dtype), parity.to_gpu(W, dtype), parity.to_gpu(b, "fp32")
    o = orc.encode_topk(x[0], W[0], b[0], k, dtype)
    for ids, vals in (s3.sae_encode_topk(xg, Wg, bg, k), unsplit(s3, xg, Wg, bg, k)):
        torch.cuda.synchronize()
        assert np.array_equal(ids[0].cpu().numpy(), o["ids"]) and np.array_equal(vals[0].cpu().numpy(), o["vals"])


@pytest.mark.parametrize("heads,T,n_feat,k", [
    (2, 4, 32768, 128),      # as many ranges as there are chunks
    (1, 4096, 1024, 128),    # 128 token tiles: two ranges
    (1, 4097, 640, 33),      # 129 tiles: one range
    (8, 1024, 384, 64),      # 256 tiles, the most that are taken here
    (1, 8193, 384, 7),       # one more: the fast kernel
    (260, 3, 128, 1),
])
def test_bf16_128_calls_of_few_tokens_match_the_fast_kernel(heads, T, n_feat, k):
    """A plain call of few tokens runs tiled, a streamed one on the fast kernel: both accumulate alike, so equal bits."""
    import torch
    import paper_2601_17702_amd as s3
    g = torch.Generator(device="cuda").manual_seed(heads + T + n_feat + k)
    x = torch.randn(heads, T, 128, generator=g, device="cuda").bfloat16()
    W = (torch.randn(heads, n_feat, 128, generator=g, device="cuda") / 11).bfloat16()
    b = 0.1 * torch.randn(heads, n_feat, generator=g, device="cuda")
    ids0, vals0 = s3.sae_encode_topk_stream(x, W, b, k, s3.new_tau_hint(heads))
    for ids, vals in (s3.sae_encode_topk(x, W, b, k), unsplit(s3, x, W, b, k)):
        torch.cuda.synchronize()
        assert torch.equal(ids, ids0) and torch.equal(vals, vals0)


@pytest.mark.parametrize("dtype,d,heads,T,n_feat,k,live", [
    ("bf16", 128, 2, 3, 512, 64, 63),      # one element short of a full row; two ranges
    ("bf16", 128, 1, 1, 640, 128, 0),      # no element at all; lists of 256
    ("bf16", 64, 1, 33, 300, 65, 64),
    ("fp32", 128, 1, 5, 16, 16, 5),        # every feature is in the row
    ("fp32", 256, 3, 2, 1025, 2, 1),
])
def test_rows_with_fewer_than_k_elements_are_whole(dtype, d, heads, T, n_feat, k, live):
    """A bias of -inf on all but `live` features: they come first, then the lowest other ids with value 0, as in a stable sort
    of the pre-activations; a token of NaN has ids 0 .. k - 1.  Small integers, so the sums are exact."""
    import torch
    import paper_2601_17702_amd as s3
    rng = np.random.default_rng(n_feat + k)
    xf = rng.integers(-2, 3, (heads, T, d)).astype(np.float32)
    Wf = rng.integers(-2, 3, (heads, n_feat, d)).astype(np.float32)
    b = np.full((heads, n_feat), -np.inf, np.float32)
    for h in range(heads):
        b[h, rng.permutation(n_feat)[:live]] = 500.0
    xf[0, T - 1, d // 2] = np.nan
    z = np.einsum("htd,hfd->htf", xf, Wf) + b[:, None]
    z = np.where(np.isnan(z), -np.inf, z)
    want = np.argsort(-z, axis=2, kind="stable")[:, :, :k]
    want_v = np.maximum(np.take_along_axis(z, want, axis=2), 0)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    xg, Wg, bg = torch.from_numpy(xf).cuda().to(dt), torch.from_numpy(Wf).cuda().to(dt), torch.from_numpy(b).cuda()
    ids = torch.full((heads, T, k), -7, dtype=torch.int32, device="cuda")
    vals = torch.full((heads, T, k), -7.0, device="cuda")
    s3.sae_encode_topk(xg, Wg, bg, k, ids, vals)
    torch.cuda.synchronize()
    assert np.array_equal(ids.cpu().numpy(), want) and np.array_equal(vals.cpu().numpy(), want_v)


@pytest.mark.parametrize("heads,T", [(1, (1 << 28) + 33), ((1 << 23) + 5, 1), (3, (1 << 27) + 32)])
def test_more_workgroups_than_one_launch_holds(heads, T):
    """Over 2^23 token tiles: more than 2^32 threads.  All rows are zero, so their id is the largest bias of the head, but for
    some at the ends and around the middle; those must come out as in calls of their own."""
    import torch
    import paper_2601_17702_amd as s3
    d, n_feat = 64, 8
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of device memory")
    g = torch.Generator(device="cuda").manual_seed(5)
    W = torch.randn(heads, n_feat, d, generator=g, device="cuda", dtype=torch.bfloat16)
    b = torch.rand(heads, n_feat, generator=g, device="cuda")
    x = torch.zeros(heads, T, d, dtype=torch.bfloat16, device="cuda")
    flat = x.view(heads * T, d)
    n = heads * T
    rows = torch.cat([torch.arange(c, c + 70, device="cuda") for c in (0, n // 4 - 35, n // 2 - 35, n // 2 + n // 4 - 35, n - 70)])
    flat[rows] = torch.randn(len(rows), d, generator=g, device="cuda").bfloat16()
    ids, vals = s3.sae_encode_topk(x, W, b, 1)
    of = rows // T
    ids1, vals1 = s3.sae_encode_topk(flat[rows][:, None].contiguous(), W[of], b[of], 1)      # each row as a head of one token
    torch.cuda.synchronize()
    assert torch.equal(ids.view(-1)[rows], ids1.view(-1)) and torch.equal(vals.view(-1)[rows], vals1.view(-1))
    top_v, top = b.max(dim=1)
    plain = torch.ones(n, dtype=torch.bool, device="cuda")
    plain[rows] = False
    plain = plain.view(heads, T)
    assert not bool(((ids[:, :, 0] != top[:, None]) & plain).any()) and not bool(((vals[:, :, 0] != top_v[:, None]) & plain).any())
