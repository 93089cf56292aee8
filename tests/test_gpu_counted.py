"""lkv_score_counted / lkv_select_counted: the scoring launch counts the first-level digits of the top-k's radix
descent (the top 11 bits of every score's order-preserving key) and the top-k starts from those counts.  Scores,
kept indices and offsets must equal those of lkv_score / lkv_select bit for bit (and hence the oracle's top-k on
the GPU's scores); the counts must be the histogram of the written scores, and zero again after the top-k."""
import numpy as np
import pytest
import torch

from oracle import lkv_oracle as O
from paper_2605_06676_amd import lkv
from paper_2605_06676_amd import workloads as W

import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = lkv.Context(0)
    yield c
    c.close()


def _case(ctx, w, Ts, seed=0, budgets=None):
    Ks, Vs, Qs, Bs = [], [], [], []
    for s, T in enumerate(Ts):
        K, V = W.draw_kv(w, T, s, seed)
        Ks.append(K); Vs.append(V); Qs.append(W.draw_q(w, s, seed))
        Bs.append(W.draw_budgets(w, T, s, seed) if budgets is None else budgets[s])
    sc = W.draw_scorer(w, seed)
    run = G.GpuRun(ctx, Ks, Vs, Qs, sc, Bs, w.Hq)
    run.run_all()
    return run, (Ks, Vs, Qs, sc, Bs)


def _counted_equals_plain(ctx, run, what):
    c = run.cache
    counts = torch.full((c.n_segments, 2048), 0x55555555, dtype=torch.int32, device="cuda")
    lkv.lkv_clear_counts(ctx, counts, c.n_segments)
    torch.cuda.synchronize()
    assert int(counts.abs().max()) == 0, f"{what}: lkv_clear_counts"
    scores = [torch.full_like(s, float("nan")) for s in run.scores]
    idx = torch.full_like(run.idx, -5)
    offsets = torch.full_like(run.offsets, -5)
    for rep in range(2):      # the second pair starts from the counters the first one left behind
        lkv.lkv_score_counted(ctx, c, run.scorer, scores, counts)
        torch.cuda.synchronize()
        seg = 0
        for s in range(c.n_seq):
            assert torch.equal(scores[s].view(torch.int32), run.scores[s].view(torch.int32)), \
                f"{what}: scores of sequence {s} differ from lkv_score"
            u = scores[s].cpu().numpy().reshape(c.L * c.H, -1)
            got = counts[seg:seg + c.L * c.H].cpu().numpy()
            for j in range(c.L * c.H):
                want = np.bincount((O.order_key(u[j]) >> np.uint32(21)).astype(np.int64), minlength=2048)
                assert np.array_equal(got[j], want), f"{what}: counts of sequence {s} head {j}"
            seg += c.L * c.H
        idx.fill_(-5); offsets.fill_(-5)
        lkv.lkv_select_counted(ctx, c, scores, run.budgets, counts, idx, offsets)
        torch.cuda.synchronize()
        assert torch.equal(offsets, run.offsets), f"{what}: offsets"
        assert torch.equal(idx[:run.total], run.idx[:run.total]), f"{what}: kept indices differ from lkv_select (pass {rep})"
        assert int(counts.abs().max()) == 0, f"{what}: counters not left zero"


@pytest.mark.parametrize("scorer,hidden,act,per_head", [("linear", 0, "gelu", False), ("mlp", 64, "gelu", False),
                                                       ("mlp", 32, "silu", True), ("mlp", 128, "silu", True),
                                                       ("mlp", 96, "gelu", False)])
@pytest.mark.parametrize("T", [1, 300, 5000, 34304, 40000])
def test_counted_path_equals_plain_path(ctx, scorer, hidden, act, per_head, T):
    w = W.scaled(W.CONFIGS[0], L=2, H=3, Hq=6, scorer=scorer, hidden=hidden, act=act, per_head=per_head, b_min=min(4, T), R=0.2)
    budgets = [np.array([[1, 0, 1], [0, 1, 1]], dtype=np.int32)] if T == 1 else None
    run, (Ks, Vs, Qs, sc, Bs) = _case(ctx, w, [T], seed=T % 7, budgets=budgets)
    G.check_against_oracle(run, Ks, Vs, Qs, sc, Bs, f"{scorer}-{hidden} T={T}")
    _counted_equals_plain(ctx, run, f"{scorer}-{hidden} T={T}")


def test_counted_path_long_heads_of_the_131072_token_workload(ctx):
    w = W.scaled(W.CONFIGS[2], L=1, H=2, Hq=8)
    run, _ = _case(ctx, w, [131072], seed=3)
    _counted_equals_plain(ctx, run, "T=131072")


def test_counted_path_many_sequences_and_degenerate_budgets(ctx):
    # 40 sequences: two launches of every kernel; budgets 0 and T among them (their counters must be zeroed too)
    rng = np.random.default_rng(5)
    Ts = [int(t) for t in rng.integers(30, 500, size=40)]
    Ts[3] = 36000
    w = W.scaled(W.CONFIGS[0], n_seq=40, L=1, H=2, Hq=4, scorer="mlp", hidden=48, act="silu", b_min=2)
    budgets = []
    for s, T in enumerate(Ts):
        b = W.draw_budgets(w, T, s, 8)
        if s % 5 == 0:
            b[0, 0] = 0
        if s % 7 == 0:
            b[0, 1] = T
        budgets.append(b)
    run, (Ks, Vs, Qs, sc, Bs) = _case(ctx, w, Ts, seed=8, budgets=budgets)
    G.check_against_oracle(run, Ks, Vs, Qs, sc, Bs, "40 sequences")
    _counted_equals_plain(ctx, run, "40 sequences")


def test_counted_path_with_special_scores(ctx):
    # a linear scorer that reads key channel 0 (weight one-hot, bias 0) makes the scores any bf16 pattern we like:
    # NaN, infinities, zeros and long runs of ties; the counted top-k must agree with the plain one and the oracle
    T = 41000
    w = W.scaled(W.CONFIGS[0], L=1, H=2, Hq=4, b_min=8)
    K, V = W.draw_kv(w, T, 0, 4)
    rng = np.random.default_rng(12)
    col = W.bf16_bits_to_f32(K[0, :, :, 0]).copy()
    col[0, ::7] = np.float32(0.5)                      # ties across the threshold
    col[0, 5:4000:11] = np.float32("nan")
    col[0, 9:9000:13] = np.float32("inf")
    col[1, :] = np.float32(0.0)
    col[1, ::3] = np.float32("-inf")
    col[1, 1::3] = rng.choice(np.array([1.0, 2.0, -1.0], dtype=np.float32), size=col[1, 1::3].size)
    K[0, :, :, 0] = W.f32_to_bf16_bits(col)
    sc = W.draw_scorer(w, 4)
    sc["w1"][:] = 0
    sc["w1"][:, :, 0] = W.f32_to_bf16_bits(np.float32(1.0))
    sc["b1"][:] = 0
    B = np.array([[12000, 20000]], dtype=np.int32)
    run = G.GpuRun(ctx, [K], [V], [W.draw_q(w, 0, 4)], sc, [B], w.Hq)
    run.score(); run.select()
    torch.cuda.synchronize()
    u = run.scores[0].cpu().numpy()
    assert np.isnan(u[0, 0]).sum() > 300 and np.isposinf(u[0, 0]).sum() > 300
    idx_ref, off_ref = O.select_all(u, B)
    assert np.array_equal(run.idx.cpu().numpy()[:int(off_ref[-1])], idx_ref)
    _counted_equals_plain(ctx, run, "special scores")


@pytest.mark.parametrize("scorer,hidden", [("linear", 0), ("mlp", 64), ("mlp", 128)])
def test_layer_by_layer_eviction_with_counts(ctx, scorer, hidden):
    w = W.scaled(W.CONFIGS[0], n_seq=2, L=5, H=3, Hq=6, scorer=scorer, hidden=hidden, act="silu", per_head=hidden == 128, b_min=4)
    Ts = [36000, 700]
    Ks, Vs, Qs, Bs = [], [], [], []
    for s, T in enumerate(Ts):
        K, V = W.draw_kv(w, T, s, 6)
        Ks.append(K); Vs.append(V); Qs.append(W.draw_q(w, s, 6)); Bs.append(W.draw_budgets(w, T, s, 6))
    sc = W.draw_scorer(w, 6)
    whole = G.GpuRun(ctx, Ks, Vs, Qs, sc, Bs, w.Hq)
    whole.run_all()
    for m in (1, 2):
        lay = G.LayerwiseRun(ctx, Ks, Vs, Qs, sc, Bs, w.Hq)
        counts = torch.zeros((lay.cache.n_segments, 2048), dtype=torch.int32, device="cuda")
        lay.evict_layerwise(order=[4, 0, 2] if m == 2 else [3, 1, 4, 0, 2], layers_per_call=m, counts=counts)
        lay.decode()
        torch.cuda.synchronize()
        n = whole.total
        assert torch.equal(lay.offsets, whole.offsets) and torch.equal(lay.idx[:n], whole.idx[:n])
        assert torch.equal(lay.kp[:n].view(torch.int16), whole.kp[:n].view(torch.int16))
        assert torch.equal(lay.vp[:n].view(torch.int16), whole.vp[:n].view(torch.int16))
        assert torch.equal(lay.out, whole.out)
        assert int(counts.abs().max()) == 0


def test_counted_calls_report_argument_errors(ctx):
    w = W.scaled(W.CONFIGS[0], L=1, H=2, Hq=4, b_min=4)
    run, _ = _case(ctx, w, [256])
    lib = lkv.load_library()
    with pytest.raises(lkv.LkvError) as e:
        ctx._check(lib.lkv_clear_counts(ctx.h, None, 2, None))
    assert e.value.status == 1
    counts = torch.zeros((2, 2048), dtype=torch.int32, device="cuda")
    with pytest.raises(lkv.LkvError) as e:
        ctx._check(lib.lkv_clear_counts(ctx.h, counts.data_ptr() + 4, 2, None))
    assert e.value.status == 1
    assert lkv.lkv_counts_bytes(3) == 3 * 2048 * 4 and lkv.lkv_counts_bytes(0) == 0


def _layerwise_equals_whole(ctx, w, Ts, seed, split, Ks=None, Vs=None, sc=None, Bs=None, orders=((1, None),)):
    if Ks is None:
        Ks, Vs, Bs = [], [], []
        for s, T in enumerate(Ts):
            K, V = W.draw_kv(w, T, s, seed)
            Ks.append(K); Vs.append(V); Bs.append(W.draw_budgets(w, T, s, seed))
        sc = W.draw_scorer(w, seed)
    Qs = [W.draw_q(w, s, seed) for s in range(len(Ts))]
    whole = G.GpuRun(ctx, Ks, Vs, Qs, sc, Bs, w.Hq)
    whole.run_all()
    idx_ref = []
    for s in range(len(Ts)):
        idx_ref.append(O.select_all(whole.scores[s].cpu().numpy(), np.asarray(Bs[s]).reshape(w.L, w.H))[0])
    assert np.array_equal(whole.idx.cpu().numpy()[:whole.total], np.concatenate(idx_ref))
    n_seg = whole.cache.n_segments
    nbytes = lkv.lkv_counts_bytes_split(n_seg, max(Ts)) if split else lkv.lkv_counts_bytes(n_seg)
    for m, order in orders:
        lay = G.LayerwiseRun(ctx, Ks, Vs, Qs, sc, Bs, w.Hq)
        counts = torch.full((nbytes // 4,), 0x33333333, dtype=torch.int32, device="cuda")      # the bitmaps need no clearing
        lkv.lkv_clear_counts(ctx, counts, n_seg)
        lay.evict_layerwise(order=order, layers_per_call=m, counts=counts)
        lay.decode()
        torch.cuda.synchronize()
        n = whole.total
        assert torch.equal(lay.offsets, whole.offsets) and torch.equal(lay.idx[:n], whole.idx[:n]), f"m={m}: indices"
        assert torch.equal(lay.kp[:n].view(torch.int16), whole.kp[:n].view(torch.int16))
        assert torch.equal(lay.vp[:n].view(torch.int16), whole.vp[:n].view(torch.int16))
        assert torch.equal(lay.out, whole.out)
        assert int(counts[:n_seg * 2048].abs().max()) == 0, "counters not left zero"


@pytest.mark.parametrize("scorer,hidden,T", [("mlp", 64, 40000), ("linear", 0, 70001), ("mlp", 128, 34305), ("mlp", 32, 131072)])
def test_long_heads_split_over_several_workgroups(ctx, scorer, hidden, T):
    # one layer at a time over heads too long for the top-k's registers, with room for the bitmaps behind the
    # counters: every head's pass over the scores is split over several workgroups; the result must not change
    L, H = (1, 2) if T > 100000 else (3, 2)
    w = W.scaled(W.CONFIGS[0], L=L, H=H, Hq=2 * H, scorer=scorer, hidden=hidden, act="gelu", per_head=hidden == 128, b_min=16, R=0.1)
    _layerwise_equals_whole(ctx, w, [T], seed=3, split=True, orders=((1, None), (2, None)) if L > 1 else ((1, None),))


def test_split_route_with_two_long_sequences_and_without_room_for_the_bitmaps(ctx):
    w = W.scaled(W.CONFIGS[0], n_seq=2, L=2, H=2, Hq=4, scorer="mlp", hidden=48, act="silu", b_min=8)
    _layerwise_equals_whole(ctx, w, [36001, 50000], seed=5, split=True)
    _layerwise_equals_whole(ctx, w, [36001, 50000], seed=5, split=False)      # counters only: the unsplit counted route


def test_split_route_falls_back_when_the_undecided_bin_is_too_full(ctx):
    # scores of one head crowd into one first-level bin ([1, 1.25): one value of the top 11 key bits): more
    # candidates than the top-k lists, so that head takes the unsplit route inside the same launch; the other head
    # is split as usual.  A one-hot linear scorer makes the scores key channel 0.
    T = 45000
    w = W.scaled(W.CONFIGS[0], L=2, H=2, Hq=4, b_min=8)
    K, V = W.draw_kv(w, T, 0, 9)
    rng = np.random.default_rng(9)
    col = W.bf16_bits_to_f32(K[:, :, :, 0]).copy()                           # [L, H, T]
    col[0, 0, :] = 1.0 + rng.integers(0, 32, size=T).astype(np.float32) / 128.0     # 32 bf16 values in [1, 1.25)
    col[1, 1, : T // 2] = np.float32(3.0)                                    # a long run of ties in the other layer
    K[:, :, :, 0] = W.f32_to_bf16_bits(col)
    sc = W.draw_scorer(w, 9)
    sc["w1"][:] = 0
    sc["w1"][:, :, 0] = W.f32_to_bf16_bits(np.float32(1.0))
    sc["b1"][:] = 0
    B = np.array([[20000, 3000], [9000, 30000]], dtype=np.int32)
    _layerwise_equals_whole(ctx, w, [T], seed=9, split=True, Ks=[K], Vs=[V], sc=sc, Bs=[B])


def test_counts_buffer_too_small_is_an_error(ctx):
    w = W.scaled(W.CONFIGS[0], L=2, H=2, Hq=4, b_min=4)
    K, V = W.draw_kv(w, 300, 0, 1)
    run = G.LayerwiseRun(ctx, [K], [V], [W.draw_q(w, 0, 1)], W.draw_scorer(w, 1), [W.draw_budgets(w, 300, 0, 1)], w.Hq)
    lkv.lkv_plan_offsets(ctx, run.budgets, run.offsets)
    view = lkv.Cache([run.k[0][0:1]], [run.v[0][0:1]], w.Hq)
    scratch = [torch.empty((1, w.H, 300), dtype=torch.float32, device="cuda")]
    small = torch.zeros((3 * 2048,), dtype=torch.int32, device="cuda")          # 4 segments need 4 x 2048 counters
    with pytest.raises(lkv.LkvError) as e:
        lkv.lkv_evict_layer(ctx, view, 0, w.L, run.scorer, run.budgets, run.offsets, scratch, run.idx, run.kp, run.vp, counts=small)
    assert e.value.status == 3
    assert lkv.lkv_counts_bytes_split(4, 100) == 4 * 2048 * 4 + 4 * 2 * 4 * 4
    torch.cuda.synchronize()


@pytest.mark.parametrize("T", [34817, 40000, 327680, 327681])
def test_counts_of_other_scores_write_no_index_past_a_segment(ctx, T):
    # a caller's error: the counters counted scores below zero, the scores selected from are above it, so every token lies
    # above the bin found; what is kept means nothing then, but each segment gets as many indices as its budget
    K = torch.zeros((1, 2, T, 128), dtype=torch.bfloat16, device="cuda")
    cache = lkv.Cache([K], [K], 2)
    scorer = {"kind": "linear", "act": "silu", "hidden": 0, "per_head": False, "w2": None, "b2": None,
              "w1": torch.zeros((1, 256), dtype=torch.bfloat16, device="cuda"), "b1": torch.full((1,), -3.0, device="cuda")}
    counts = torch.zeros((2, 2048), dtype=torch.int32, device="cuda")
    scores = torch.empty((1, 2, T), device="cuda")
    lkv.lkv_score_counted(ctx, cache, scorer, [scores], counts)
    scores.uniform_(1.0, 9.0)
    b = 500
    buffer = torch.full((2 * b + T,), -1, dtype=torch.int32, device="cuda")
    offsets = torch.empty(3, dtype=torch.int32, device="cuda")
    lkv.lkv_select_counted(ctx, cache, [scores], np.full(2, b, np.int32), counts, buffer[:2 * b], offsets)
    torch.cuda.synchronize()
    assert offsets.tolist() == [0, b, 2 * b]
    assert (buffer[2 * b:] == -1).all()
    assert (buffer[:2 * b] >= -1).all() and (buffer[:2 * b] < T).all()
    assert not counts.any()
    lkv.lkv_select(ctx, cache, [scores], np.full(2, b, np.int32), buffer[:2 * b], offsets)     # and the call itself is sound
    u = scores.cpu().numpy()[0]
    for h in range(2):
        assert np.array_equal(buffer[h * b:(h + 1) * b].cpu().numpy(), O.select(u[h], b))
