"""Decode over more than 64 segments: chunks that start at the segments, four segments' bounds to a lane (up to 128
segments, up to 256 while they are short), and flat chunks, whose pieces are shared by four waves or dealt to single ones.

Against 64 bits.  An output is a weighted mean of value rows, so its error stays below the probabilities' relative error
times the largest value: they are multiplied in two bf16 parts, 2^-18, and fp32 logits of up to 2^4 and exponentials add about
2^-19.  Four times that is allowed (one part alone: 2^-9); the log-sum-exp is an fp32 sum of fp32 exponentials."""
import numpy as np
import pytest
import torch

from paper_2605_06676_amd import lkv

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 64, 65, 127, 128, 129, 0, 256, 257, 500]


@pytest.fixture(scope="module")
def ctx():
    c = lkv.Context(0)
    yield c
    c.close()


def _skewed(n, longest, seed):
    return (longest * np.random.default_rng(seed).random(n) ** 6).astype(int).tolist()


CASES = {
    # chunks that start at the segments
    "65": (EDGES * 5, 65, 4),
    "67, long last one": (EDGES * 5, 66, 3, 4000),
    "128 skewed": (_skewed(128, 20000, 1), 128, 1),
    "127 equal": ([384] * 127, 127, 16),
    "129": (EDGES * 10, 129, 8),
    "255 skewed": (_skewed(255, 6000, 2), 255, 4),
    "256 empty but one": ([0] * 255, 255, 2, 3000),
    "256, most rows that still do": ([1536] * 256, 256, 1),
    # flat chunks
    "256, one row more": ([1536] * 255, 255, 1, 1537),
    "257": (EDGES * 19, 257, 4),
    "dozens of segments to a chunk": ([1, 0, 0, 2] * 300, 1200, 2),
    "one row each around a long one": ([1] * 200 + [2000] + [1] * 150, 351, 7),
    "long and short": (([700, 3, 40, 0, 90, 300] * 60), 360, 4),
    "512 skewed": (_skewed(512, 9000, 3), 512, 1),
    "a wave's share and more": ([1024, 1025, 60, 512, 513, 33] * 80, 480, 16),
}


def _lengths(name):
    base, n, g, *last = CASES[name]
    return base[:n] + last, g


def _check(got, got_lse, q, k, v, starts, lengths):
    assert torch.isfinite(got).all()
    vmax = float(v.abs().max())
    for s, (at, m) in enumerate(zip(starts, lengths)):
        if m == 0:
            assert (got[s] == 0).all() and torch.isneginf(got_lse[s]).all(), s
            continue
        x = q[s] @ k[at:at + m].T * 128 ** -0.5
        err = float((got[s] - torch.softmax(x, dim=1) @ v[at:at + m]).abs().max())
        assert err <= 2.0 ** -16 * vmax, (s, m, err)
        assert float((got_lse[s] - torch.logsumexp(x, dim=1)).abs().max()) <= 2.0 ** -16, (s, m)


@pytest.mark.parametrize("spare", [0, 5], ids=["packed", "grown"])
@pytest.mark.parametrize("name", CASES)
def test_pieces_of_many_segments(ctx, name, spare):
    lengths, g = _lengths(name)
    if spare and lengths[0] == 1536:
        pytest.skip("the rows that a launch may hold count the spare ones")
    n = len(lengths)
    caps = [m + spare for m in lengths]
    total = sum(caps)
    gen = torch.Generator(device="cuda").manual_seed(total)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, k, v = normal(1, 1, n * g, 128), normal(total, 128), normal(total, 128)
    k[total // 2:] *= 2    # the maxima of the pieces differ
    starts = np.concatenate([[0], np.cumsum(caps)])
    offsets = torch.from_numpy(starts.astype(np.int32)).cuda()
    out = torch.full((1, 1, n * g, 128), float("nan"), device="cuda")
    lse = torch.full((1, 1, n * g), float("nan"), device="cuda")
    ws = torch.full((lkv.lkv_decode_workspace_bytes(n, total, n * g, n),), 255, dtype=torch.uint8, device="cuda")
    qd, kd, vd = q.cpu().double().view(n, g, 128), k.cpu().double(), v.cpu().double()
    if spare:
        for at, m in zip(starts, lengths):      # rows that are not in use hold what no result may show
            k[at + m:at + m + spare] = float("nan")
            v[at + m:at + m + spare] = float("nan")
        used = torch.tensor(lengths, dtype=torch.int32, device="cuda")
        lkv.lkv_decode_attn_grown(ctx, 1, 1, n, n * g, 128, q, k, v, offsets, used, total, 128 ** -0.5, out, lse, ws)
    else:
        lkv.lkv_decode_attn(ctx, 1, 1, n, n * g, 128, q, k, v, offsets, total, 128 ** -0.5, out, lse, ws)
    _check(out.cpu().double().view(n, g, 128), lse.cpu().double().view(n, g), qd, kd, vd, starts, lengths)


@pytest.mark.parametrize("heads,T", [(66, 70), (130, 200), (256, 129), (260, 100)])
def test_masked_decode_over_many_heads(ctx, heads, T):
    gen = torch.Generator(device="cuda").manual_seed(heads)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    L, H = 2, heads // 2
    k, v, q = normal(L, H, T, 128), normal(L, H, T, 128), normal(1, L, H * 2, 128)
    m = torch.rand(L, H, T, device="cuda", generator=gen)
    m[m < 0.3] = 0
    m[1, 3] = 0                                  # a head without any weight
    cache = lkv.Cache([k], [v], H * 2)
    out, lse = torch.empty(1, L, H * 2, 128, device="cuda"), torch.empty(1, L, H * 2, device="cuda")
    ws = torch.empty(lkv.lkv_masked_decode_workspace_bytes(cache), dtype=torch.uint8, device="cuda")
    lkv.lkv_masked_decode_attn(ctx, cache, q, [m], 128 ** -0.5, out, lse, ws)
    got, got_lse = out.cpu().double().view(heads, 2, 128), lse.cpu().double().view(heads, 2)
    kd, vd, md, qd = (x.cpu().double().reshape(heads, *x.shape[2:]) if x is not q else x.cpu().double().view(heads, 2, 128)
                      for x in (k, v, m, q))
    vmax = float(vd.abs().max())
    for s in range(heads):
        if float(md[s].sum()) == 0:
            assert (got[s] == 0).all() and torch.isneginf(got_lse[s]).all()
            continue
        x = qd[s] @ kd[s].T * 128 ** -0.5 + torch.log(md[s])
        assert float((got[s] - torch.softmax(x, dim=1) @ vd[s]).abs().max()) <= 2.0 ** -16 * vmax, s
        assert float((got_lse[s] - torch.logsumexp(x, dim=1)).abs().max()) <= 2.0 ** -16, s


@pytest.mark.parametrize("n", [8, 100, 300])
def test_infinite_values_stay_infinite(ctx, n):
    """A value row with an infinite channel: the second part of its probability is 0 or negative and is not multiplied
    from there on, so the channel is infinite, not NaN, and the others keep at least one part's digits."""
    m, g = 300, 2
    gen = torch.Generator(device="cuda").manual_seed(n)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, k, v = normal(1, 1, n * g, 128), normal(n * m, 128), normal(n * m, 128)
    offsets = torch.arange(0, n * m + 1, m, dtype=torch.int32, device="cuda")
    at = m * (n // 2) + 200
    ref = v.cpu().double()
    v[at, 5], v[at, 9] = float("inf"), float("-inf")
    out = torch.empty(1, 1, n * g, 128, device="cuda")
    ws = torch.empty(lkv.lkv_decode_workspace_bytes(n, n * m, n * g, n), dtype=torch.uint8, device="cuda")
    lkv.lkv_decode_attn(ctx, 1, 1, n, n * g, 128, q, k, v, offsets, n * m, 128 ** -0.5, out, None, ws)
    got = out.cpu().double().view(n, g, 128)
    assert (got[n // 2, :, 5] == float("inf")).all() and (got[n // 2, :, 9] == float("-inf")).all()
    p = torch.softmax(torch.einsum("sgd,smd->sgm", q.cpu().double().view(n, g, 128), k.cpu().double().view(n, m, 128)) * 128 ** -0.5, dim=2)
    want = torch.einsum("sgm,smd->sgd", p, ref.view(n, m, 128))
    want[n // 2, :, [5, 9]] = got[n // 2, :, [5, 9]] = 0
    assert (got - want).abs().max() <= 2.0 ** -8 * ref.abs().max()
