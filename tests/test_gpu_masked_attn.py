"""GPU parity of the training-time attention with a multiplicative mask (App. B) against the
fp64 oracle, through the C ABI.  The bound on the outputs is the decode bound (2e-2 of the
output scale of the query row); the log-normaliser is held to 1e-3 absolute."""
import numpy as np
import pytest
import torch

from oracle import lkv_oracle as O
from oracle import masked_attn as MA
from paper_2605_06676_amd import lkv
from paper_2605_06676_amd import workloads as W
from tests.gpu_util import SCALE, assert_decode_close, bf16_gpu_to_bits, bits_to_bf16_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = lkv.Context(0)
    yield c
    c.close()


def run_forward(ctx, q, k, v, m):
    tq, tk, tv = (bits_to_bf16_gpu(x) for x in (q, k, v))
    tm = torch.from_numpy(m).cuda()
    o = torch.full(tq.shape, float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full(tq.shape[:2], float("nan"), dtype=torch.float32, device="cuda")
    lkv.lkv_masked_attn_forward(ctx, tq, tk, tv, tm, SCALE, o, lse)
    torch.cuda.synchronize()
    return o.cpu().numpy(), lse.cpu().numpy()


def check_forward(ctx, Hq, H, T, seed=0, mask=None):
    q, k, v, m, _ = W.draw_training_attention(Hq, H, T, seed)
    if mask is not None:
        m = mask(m)
    o_gpu, lse_gpu = run_forward(ctx, q, k, v, m)
    o_ref, lse_ref = MA.forward(*(O.bf16_bits_to_f64(x) for x in (q, k, v)), m, SCALE)
    return assert_decode_close(o_gpu.reshape(-1, 128), lse_gpu.reshape(-1), o_ref.reshape(-1, 128), lse_ref.reshape(-1),
                               f"Hq{Hq} H{H} T{T}")


@pytest.mark.parametrize("Hq,H,T", [(4, 2, 300), (2, 2, 1), (1, 1, 33), (4, 1, 128), (2, 1, 129), (7, 1, 257), (8, 2, 1000), (16, 1, 70), (3, 3, 64),
                                    (6, 2, 513)])
def test_forward_small(ctx, Hq, H, T):
    check_forward(ctx, Hq, H, T)


def test_forward_wide_blocks(ctx):
    # long enough for the 256-query blocks, ragged against every tile size
    check_forward(ctx, 2, 1, 8192 + 77)


def test_forward_mask_edge_cases(ctx):
    def zero_prefix(m):
        m = m.copy()
        m[:, :37] = 0.0          # the first 37 queries see no weight at all: zero output, lse = -inf
        return m

    check_forward(ctx, 4, 2, 200, mask=zero_prefix)
    check_forward(ctx, 4, 2, 200, mask=lambda m: np.ones_like(m))                       # plain causal attention
    check_forward(ctx, 4, 2, 200, mask=lambda m: (m > 0.2).astype(np.float32))   # 0/1 mask, first key kept


@pytest.mark.parametrize("T", [97, 128, 300, 641])
@pytest.mark.parametrize("factor", [6.0, 12.0, 40.0])
def test_forward_logits_that_run_away_from_the_first_keys(ctx, T, factor):
    # The references of the exponentials are set by the first 32 keys.  Keys further on scaled up leave them behind: the
    # sums against them reach up to 2^34 with factor 6, more than 2^56 with 12 and more than fp32 holds with 40.  One head
    # also has its largest logits at keys of weight 0.
    q, k, v, m, _ = W.draw_training_attention(4, 2, T, seed=5)
    kf = O.bf16_bits_to_f64(k)
    kf[:, 40:] *= factor
    k = W.f32_to_bf16_bits(kf.astype(np.float32))
    m[1, 3:20] = 0.0
    o_gpu, lse_gpu = run_forward(ctx, q, k, v, m)
    o_ref, lse_ref = MA.forward(*(O.bf16_bits_to_f64(x) for x in (q, k, v)), m, SCALE)
    assert_decode_close(o_gpu.reshape(-1, 128), lse_gpu.reshape(-1), o_ref.reshape(-1, 128), lse_ref.reshape(-1),
                        f"T{T} factor {factor}")


@pytest.mark.parametrize("Hq,H,T", [(4, 2, 1), (4, 2, 31), (2, 1, 128), (4, 1, 129), (4, 2, 700)])
def test_forward_first_queries_keep_more_digits_of_the_weights(ctx, Hq, H, T):
    # The first 128 queries multiply the weights in two bf16 parts (relative error 2^-18 each), the others in one (2^-9).
    # An output is a weighted mean of value rows, so its error stays below the weights' times the largest value, and what
    # fp32 logits of up to 2^5 and exponentials add is 2^-19 of it each; twice to four times that are allowed.
    q, k, v, m, _ = W.draw_training_attention(Hq, H, T, seed=8)
    o_gpu, _ = run_forward(ctx, q, k, v, m)
    qf, kf, vf = (O.bf16_bits_to_f64(x) for x in (q, k, v))
    o_ref, _ = MA.forward(qf, kf, vf, m, SCALE)
    err = np.abs(o_gpu - o_ref).max(axis=(0, 2)) / np.abs(vf).max()
    assert err[:128].max() <= 2.0 ** -16, err[:128].max()
    assert T <= 128 or err[128:].max() <= 2.0 ** -8, err[128:].max()


def _log2_sum_against_first_keys(q, k, m):
    """Largest log2 over all queries of sum_j 2^(x_ij - ref_i) m_j, ref_i the largest x_ij among the first 32 keys."""
    G, most = q.shape[0] // k.shape[0], -np.inf
    for hq in range(q.shape[0]):
        x = q[hq] @ k[hq // G].T * SCALE * np.log2(np.e)
        x[np.triu_indices_from(x, 1)] = -np.inf
        y = x + np.log2(np.maximum(m[hq // G].astype(np.float64), 1e-300))[None, :] - x[:, :32].max(axis=1, keepdims=True)
        top = y.max(axis=1)
        most = max(most, (top + np.log2(np.exp2(y - top[:, None]).sum(axis=1))).max())
    return most


@pytest.mark.parametrize("T", [300, 641])
@pytest.mark.parametrize("reach,v_scale", [(15, 1.0), (25, 1.0), (118, 1.0), (135, 1.0), (300, 1.0), (40, 2.0 ** 100)])
def test_forward_either_side_of_the_limits_of_the_sums(ctx, T, reach, v_scale):
    # A wave that finds a lane's sum (a quarter of a query's, 2^2 less at most) above 2^20 moves the references of its
    # queries; where a sum, or its product with the value rows, leaves fp32's range (2^128), the block starts over with
    # references that follow the maxima.  Keys from 40 on are scaled so that the largest sum comes out at 2^reach, within
    # three binary orders of what bf16 keys can be set to.
    q, k, v, m, _ = W.draw_training_attention(2, 1, T, seed=6)
    qf, kf = O.bf16_bits_to_f64(q), O.bf16_bits_to_f64(k)

    def scaled(factor):
        x = kf.copy()
        x[:, 40:] *= factor
        return W.f32_to_bf16_bits(x.astype(np.float32))

    lo, hi = 1.0, 200.0
    for _ in range(20):
        mid = np.sqrt(lo * hi)
        if _log2_sum_against_first_keys(qf, O.bf16_bits_to_f64(scaled(mid)), m) < reach: lo = mid
        else: hi = mid
    k = scaled(lo)
    assert abs(_log2_sum_against_first_keys(qf, O.bf16_bits_to_f64(k), m) - reach) < 3
    v = W.f32_to_bf16_bits((O.bf16_bits_to_f64(v) * v_scale).astype(np.float32))
    o_gpu, lse_gpu = run_forward(ctx, q, k, v, m)
    o_ref, lse_ref = MA.forward(qf, O.bf16_bits_to_f64(k), O.bf16_bits_to_f64(v), m, SCALE)
    assert_decode_close(o_gpu.reshape(-1, 128), lse_gpu.reshape(-1), o_ref.reshape(-1, 128), lse_ref.reshape(-1),
                        f"T{T} reach {reach} v {v_scale:g}")


def test_forward_rejects_bad_arguments(ctx):
    q, k, v, m, _ = W.draw_training_attention(4, 2, 64)
    tq, tk, tv = (bits_to_bf16_gpu(x) for x in (q, k, v))
    tm = torch.from_numpy(m).cuda()
    o = torch.empty(tq.shape, dtype=torch.float32, device="cuda")
    lse = torch.empty(tq.shape[:2], dtype=torch.float32, device="cuda")
    with pytest.raises(lkv.LkvError):
        lkv.lkv_masked_attn_forward(ctx, tq, tk[:1].repeat(3, 1, 1), tv, tm, SCALE, o, lse)   # 4 query heads, 3 KV heads
    with pytest.raises(lkv.LkvError):
        lkv.lkv_masked_attn_forward(ctx, tq, tk, tv, tm, 0.0, o, lse)
    with pytest.raises(lkv.LkvError):
        lkv.lkv_masked_attn_forward(ctx, tq, tk, tv, None, SCALE, o, lse)
    with pytest.raises(lkv.LkvError):
        lkv.lkv_masked_attn_forward(ctx, tq[:, :, :64].contiguous(), tk, tv, tm, SCALE, o, lse)   # head_dim 64


# ---- backward -------------------------------------------------------------------------------------
# Every gradient element is an fp32 sum of products in which one factor (P or dS) was rounded to bf16 on
# its way through the matrix cores (relative error up to 2^-9).  On top of that the per-query quantities the
# backward pass takes from the forward one (o_i in D_i = dO_i . o_i, and lse_i) carry the forward pass's own
# rounding of P, and an error dD_i enters every dS_ij of the row as p_ij dD_i whatever the size of the
# row's own gradient (the second query has two keys whose dS cancel: its dQ is small, the inherited error
# is not).  Hence a relative and an absolute part: per row, max error <= 2e-2 * (scale of the row: the
# larger of its biggest entry and its rms) + 2e-3 * (rms of the whole gradient tensor).
GRAD_RTOL = 2e-2
GRAD_ATOL_OF_RMS = 2e-3


def assert_rows_close(got, ref, what):
    ref = ref.reshape(-1, ref.shape[-1]).astype(np.float64)
    got = got.reshape(ref.shape).astype(np.float64)
    assert np.isfinite(got).all(), f"{what}: non-finite values"
    err = np.abs(got - ref).max(axis=-1)
    scale = np.maximum(np.abs(ref).max(axis=-1), np.sqrt((ref ** 2).mean(axis=-1)))
    if not np.any(ref):
        # a gradient that vanishes identically (a single key: dS = 0) comes out at the rounding level of
        # o = (p v) * (1 / l); the inputs are N(0, 1), so 1e-4 is far below any real gradient
        assert err.max() <= 1e-4, f"{what}: a gradient that must vanish is {err.max():.3g}"
        return
    tol = GRAD_RTOL * scale + GRAD_ATOL_OF_RMS * np.sqrt((ref ** 2).mean())
    bad = err > tol
    assert not bad.any(), f"{what}: {bad.sum()} rows out of tolerance, worst ratio {(err / tol).max():.3g}"


def run_backward(ctx, q, k, v, m, d_o):
    tq, tk, tv, tg = (bits_to_bf16_gpu(x) for x in (q, k, v, d_o))
    tm = torch.from_numpy(m).cuda()
    o = torch.empty(tq.shape, dtype=torch.float32, device="cuda")
    lse = torch.empty(tq.shape[:2], dtype=torch.float32, device="cuda")
    lkv.lkv_masked_attn_forward(ctx, tq, tk, tv, tm, SCALE, o, lse)
    nan = float("nan")
    dq = torch.full(tq.shape, nan, dtype=torch.float32, device="cuda")
    dk = torch.full(tk.shape, nan, dtype=torch.float32, device="cuda")
    dv = torch.full(tk.shape, nan, dtype=torch.float32, device="cuda")
    dm = torch.full(tm.shape, nan, dtype=torch.float32, device="cuda")
    ws = torch.empty(lkv.lkv_masked_attn_backward_workspace_bytes(tq.shape[0], tk.shape[0], tq.shape[1]), dtype=torch.uint8, device="cuda")
    lkv.lkv_masked_attn_backward(ctx, tq, tk, tv, tm, o, lse, tg, SCALE, dq, dk, dv, dm, ws)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in (dq, dk, dv, dm)]


def check_backward(ctx, Hq, H, T, seed=0, mask=None):
    q, k, v, m, d_o = W.draw_training_attention(Hq, H, T, seed)
    if mask is not None:
        m = mask(m)
    dq, dk, dv, dm = run_backward(ctx, q, k, v, m, d_o)
    rq, rk, rv, rm = MA.backward(*(O.bf16_bits_to_f64(x) for x in (q, k, v)), m, SCALE, O.bf16_bits_to_f64(d_o))
    tag = f"Hq{Hq} H{H} T{T}"
    assert_rows_close(dq, rq, tag + " dQ")
    assert_rows_close(dk, rk, tag + " dK")
    assert_rows_close(dv, rv, tag + " dV")
    assert_rows_close(dm, rm, tag + " dm")   # one row per KV head: the mask gradient of a head is judged as a vector


@pytest.mark.parametrize("Hq,H,T", [(4, 2, 300), (2, 2, 1), (1, 1, 33), (4, 1, 128), (2, 1, 129), (7, 1, 257), (8, 2, 1000), (16, 1, 70), (3, 3, 64),
                                    (6, 2, 513)])
def test_backward_small(ctx, Hq, H, T):
    check_backward(ctx, Hq, H, T)


@pytest.mark.parametrize("T", [2, 32, 34, 95, 96, 97, 127, 160, 161, 255, 256, 385])
def test_backward_around_the_steps_of_the_dq_pipeline(ctx, T):
    # a wave's last step of 32 keys holds its diagonal; the four waves of a block end one step after the other, and the
    # ring of key rows turns every four steps
    check_backward(ctx, 2, 1, T, seed=11)


@pytest.mark.parametrize("Hq,H,T,i", [(8, 2, 1000, 300),                       # 128 keys a block, a query head each
                                      (2, 1, 385, 130), (2, 1, 385, 384),      # and the last query, alone in its item
                                      (64, 64, 2049, 1000), (64, 64, 2049, 40)])   # 256 keys a block
@pytest.mark.parametrize("bad", ["q", "d_o", "o", "lse"])
def test_backward_reach_of_a_bad_query_row(ctx, Hq, H, T, i, bad):
    """A query row that is not finite spoils the gradients of the keys it sees.  Later keys of its own step of 32 have it
    multiplied with a weight of 0, which is finite in dV as long as dO is, and everywhere if only the normaliser is bad; keys of
    later steps never meet it, and keep every bit."""
    hq = Hq - 1
    q, k, v, m, d_o = W.draw_training_attention(Hq, H, T, seed=21)
    x = {"q": q, "k": k, "v": v, "d_o": d_o}
    x = {name: bits_to_bf16_gpu(bits) for name, bits in x.items()}
    x["m"] = torch.from_numpy(m).cuda()
    f = dict(dtype=torch.float32, device="cuda")
    x["o"], x["lse"] = torch.empty((Hq, T, 128), **f), torch.empty((Hq, T), **f)
    lkv.lkv_masked_attn_forward(ctx, x["q"], x["k"], x["v"], x["m"], SCALE, x["o"], x["lse"])
    ws = torch.empty(lkv.lkv_masked_attn_backward_workspace_bytes(Hq, H, T), dtype=torch.uint8, device="cuda")

    def backward():
        grads = [torch.full(s, 7.0, **f) for s in ((Hq, T, 128), (H, T, 128), (H, T, 128), (H, T))]
        lkv.lkv_masked_attn_backward(ctx, x["q"], x["k"], x["v"], x["m"], x["o"], x["lse"], x["d_o"], SCALE, *grads, ws)
        torch.cuda.synchronize()
        return grads

    clean = backward()
    x[bad][hq, i] = float("nan")
    got = backward()
    for g, c, name in zip(got[1:], clean[1:], ("dK", "dV", "dm")):
        if name == "dV" and bad == "o":
            assert torch.equal(g, c)          # dV has no D in it
            continue
        first = i + 1 if bad == "lse" or (name == "dV" and bad == "q") else (i // 32 + 1) * 32
        assert not torch.isfinite(g[H - 1, :i + 1]).any(), name
        spoiled = (~torch.isfinite(g[H - 1])).nonzero()[:, 0].max().item()
        assert spoiled < first, (name, spoiled)
        assert torch.equal(g[H - 1, first:], c[H - 1, first:]) and torch.equal(g[:H - 1], c[:H - 1]), name
    assert not torch.isfinite(got[0][hq, i]).any()
    got[0][hq, i] = clean[0][hq, i]
    assert torch.equal(got[0], clean[0])


def test_backward_mask_edge_cases(ctx):
    def zero_prefix(m):
        m = m.copy()
        m[:, :37] = 0.0          # 37 queries without any weight: they contribute nothing, and dm stays finite
        return m

    check_backward(ctx, 4, 2, 200, mask=zero_prefix)
    check_backward(ctx, 4, 2, 200, mask=lambda m: np.ones_like(m))
    check_backward(ctx, 4, 2, 200, mask=lambda m: (m > 0.2).astype(np.float32))


def test_backward_is_reproducible(ctx):
    # no atomics: two runs give the same bits
    q, k, v, m, d_o = W.draw_training_attention(8, 2, 777, 3)
    a = run_backward(ctx, q, k, v, m, d_o)
    b = run_backward(ctx, q, k, v, m, d_o)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_backward_rejects_small_workspace(ctx):
    q, k, v, m, d_o = W.draw_training_attention(4, 2, 64)
    tq, tk, tv, tg = (bits_to_bf16_gpu(x) for x in (q, k, v, d_o))
    tm = torch.from_numpy(m).cuda()
    o = torch.zeros(tq.shape, dtype=torch.float32, device="cuda")
    lse = torch.zeros(tq.shape[:2], dtype=torch.float32, device="cuda")
    dq = torch.empty(tq.shape, dtype=torch.float32, device="cuda")
    dk = torch.empty(tk.shape, dtype=torch.float32, device="cuda")
    dv = torch.empty_like(dk)
    dm = torch.empty_like(tm)
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    with pytest.raises(lkv.LkvError) as e:
        lkv.lkv_masked_attn_backward(ctx, tq, tk, tv, tm, o, lse, tg, SCALE, dq, dk, dv, dm, ws)
    assert e.value.status == 3


@pytest.mark.parametrize("Hq,H,T", [(32, 8, 16384), (4, 1, 131072 + 5)])
def test_full_size_sampled(ctx, Hq, H, T):
    """Llama-3.1-8B's attention shape (32 query heads, 8 KV heads) at the longest training length of
    the paper (16k tokens, App. C.2), in the launch configuration bench.py times.  Checked on what the
    oracle can compute row by row: forward rows and dQ rows of sampled queries, dK / dV / dm of the last
    keys (complete once every later query is included), and two identities that hold at any size:
    sum_j dV_j = sum_i dO_i over the group's queries (the weights of a row sum to 1) and
    sum_j m_j dm_j = 0 (scaling a head's mask changes nothing).  The second case is one GQA group over a
    context eight times longer, ragged against every tile size (index arithmetic at length)."""
    G = Hq // H
    gen = torch.Generator(device="cuda")
    gen.manual_seed(20260506)
    tq = torch.randn((Hq, T, 128), device="cuda", generator=gen).to(torch.bfloat16)
    tk = torch.randn((H, T, 128), device="cuda", generator=gen).to(torch.bfloat16)
    tv = torch.randn((H, T, 128), device="cuda", generator=gen).to(torch.bfloat16)
    tg = torch.randn((Hq, T, 128), device="cuda", generator=gen).to(torch.bfloat16)
    x = torch.rand((H, T), device="cuda", generator=gen)
    pick = torch.rand((H, T), device="cuda", generator=gen)
    tm = (x * x) * (x * x)
    tm[pick < 0.10] = 0.0
    tm[pick > 0.95] = 1.0
    tm[:, 0] = torch.clamp(tm[:, 0], min=0.25)
    o = torch.empty((Hq, T, 128), dtype=torch.float32, device="cuda")
    lse = torch.empty((Hq, T), dtype=torch.float32, device="cuda")
    lkv.lkv_masked_attn_forward(ctx, tq, tk, tv, tm, SCALE, o, lse)
    dq = torch.empty_like(o)
    dk = torch.empty((H, T, 128), dtype=torch.float32, device="cuda")
    dv = torch.empty_like(dk)
    dm = torch.empty_like(tm)
    ws = torch.empty(lkv.lkv_masked_attn_backward_workspace_bytes(Hq, H, T), dtype=torch.uint8, device="cuda")
    lkv.lkv_masked_attn_backward(ctx, tq, tk, tv, tm, o, lse, tg, SCALE, dq, dk, dv, dm, ws)
    torch.cuda.synchronize()

    # identities over everything
    dv_sum = dv.double().sum(dim=1)                                            # [H, 128]
    do_sum = tg.double().view(H, G, T, 128).sum(dim=(1, 2))
    scale_dv = tg.double().abs().view(H, G, T, 128).sum(dim=(1, 2))
    assert (dv_sum - do_sum).abs().max().item() <= 2.0 ** -9 * scale_dv.max().item()
    along = (dm.double() * tm.double()).sum(dim=1)
    assert along.abs().max().item() <= 2.0 ** -9 * (dm.double() * tm.double()).abs().sum(dim=1).max().item()

    # one KV head and its group on the host; the last `tail` queries and a few scattered ones
    tail = 150
    for h in (0, H - 1):
        heads = slice(h * G, (h + 1) * G)
        q, g = (O.bf16_bits_to_f64(bf16_gpu_to_bits(x[heads])) for x in (tq, tg))
        k, v = (O.bf16_bits_to_f64(bf16_gpu_to_bits(x[h:h + 1])) for x in (tk, tv))
        m = tm[h:h + 1].cpu().numpy()
        rows = [0, 1, 63, 64, 255, 256, 4097, 9000, T // 2 + 1] + list(range(T - tail, T))
        o_ref, lse_ref = MA.forward(q, k, v, m, SCALE, rows=rows)
        assert_decode_close(o[heads][:, rows].cpu().numpy().reshape(-1, 128), lse[heads][:, rows].cpu().numpy().reshape(-1),
                            o_ref[:, rows].reshape(-1, 128), lse_ref[:, rows].reshape(-1), f"full size head {h} forward")
        rq, rk, rv, rm = MA.backward(q, k, v, m, SCALE, g, rows=rows)
        assert_rows_close(dq[heads][:, rows].cpu().numpy(), rq[:, rows], f"full size head {h} dQ")
        keys = slice(T - tail, T)
        assert_rows_close(dk[h:h + 1, keys].cpu().numpy(), rk[:, keys], f"full size head {h} dK")
        assert_rows_close(dv[h:h + 1, keys].cpu().numpy(), rv[:, keys], f"full size head {h} dV")
        assert_rows_close(dm[h:h + 1, keys].cpu().numpy(), rm[:, keys], f"full size head {h} dm")


@pytest.mark.parametrize("Hq,H,T", [(64, 64, 2049), (128, 64, 1030), (96, 32, 2050), (128, 32, 1024)])
def test_backward_of_many_heads(ctx, Hq, H, T):
    # grids large enough for the 256-key blocks of the dK / dV kernel: unsplit, ragged against the block, the 64-query
    # items and the 32-query steps; split in two, three (every query head) and four.  First and last KV head whole.
    G = Hq // H
    q, k, v, m, d_o = W.draw_training_attention(Hq, H, T, seed=3)
    m[H - 1, :300] = 0.0                                   # and a head whose first queries see no weight at all
    dq, dk, dv, dm = run_backward(ctx, q, k, v, m, d_o)
    for x in (dq, dk, dv, dm):
        assert np.isfinite(x).all()
    for h in (0, H - 1):
        g = slice(h * G, (h + 1) * G)
        rq, rk, rv, rm = MA.backward(*(O.bf16_bits_to_f64(x) for x in (q[g], k[h:h + 1], v[h:h + 1])), m[h:h + 1], SCALE,
                                     O.bf16_bits_to_f64(d_o[g]))
        tag = f"Hq{Hq} H{H} T{T} head {h}"
        assert_rows_close(dq[g], rq, tag + " dQ")
        assert_rows_close(dk[h:h + 1], rk, tag + " dK")
        assert_rows_close(dv[h:h + 1], rv, tag + " dV")
        assert_rows_close(dm[h:h + 1], rm, tag + " dm")


@pytest.mark.parametrize("Hq,H,T", [(128, 64, 1030), (96, 32, 2050)])
def test_backward_with_a_workspace_for_whole_groups(ctx, Hq, H, T):
    # enough narrow blocks without a split: D alone is a workspace, anything between it and the full size is used as D
    # alone, and less is refused
    q, k, v, m, d_o = W.draw_training_attention(Hq, H, T, seed=4)
    tq, tk, tv, tg = (bits_to_bf16_gpu(x) for x in (q, k, v, d_o))
    tm = torch.from_numpy(m).cuda()
    f = dict(dtype=torch.float32, device="cuda")
    o, lse = torch.empty(tq.shape, **f), torch.empty(tq.shape[:2], **f)
    lkv.lkv_masked_attn_forward(ctx, tq, tk, tv, tm, SCALE, o, lse)
    full = lkv.lkv_masked_attn_backward_workspace_bytes(Hq, H, T)
    d_only = (Hq * T * 4 + 255) // 256 * 256
    assert H * ((T + 127) // 128) >= 512 and full > d_only

    def backward(n_bytes):
        ws = torch.zeros(n_bytes + 4096, dtype=torch.uint8, device="cuda")
        grads = [torch.full(s, float("nan"), **f) for s in (tq.shape, tk.shape, tk.shape, tm.shape)]
        lkv.lkv_masked_attn_backward(ctx, tq, tk, tv, tm, o, lse, tg, SCALE, *grads, ws[:n_bytes])
        torch.cuda.synchronize()
        assert not ws[n_bytes:].any()                     # nothing behind the bytes it was given
        return [x.cpu().numpy() for x in grads]

    split, whole, between = backward(full), backward(d_only), backward(full - 256)
    for a, b in zip(whole, between):
        assert np.array_equal(a, b)
    for a, b, what in zip(split, whole, ("dq", "dk", "dv", "dm")):
        assert_rows_close(a, b, what)
    with pytest.raises(lkv.LkvError) as e:
        backward(d_only - 16)
    assert e.value.status == 3


def test_random_shapes(ctx):
    # seeded draws of head counts and lengths, forward and backward, every element against the oracle
    rng = np.random.default_rng(7)
    for case in range(12):
        H = int(rng.integers(1, 4))
        G = int(rng.choice([1, 2, 3, 4, 8]))
        T = int(rng.integers(1, 420))
        check_forward(ctx, H * G, H, T, seed=100 + case)
        check_backward(ctx, H * G, H, T, seed=100 + case)
