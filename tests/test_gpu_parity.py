"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle, element by element."""
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


def _inputs(w, Ts, seed=0, budgets=None):
    K, V, Q, B = [], [], [], []
    for s, T in enumerate(Ts):
        k, v = W.draw_kv(w, T, s, seed)
        K.append(k); V.append(v); Q.append(W.draw_q(w, s, seed))
        B.append(W.draw_budgets(w, T, s, seed) if budgets is None else budgets[s])
    return K, V, Q, W.draw_scorer(w, seed), B


def _run_and_check(ctx, w, Ts, seed=0, budgets=None, what=""):
    K, V, Q, sc, B = _inputs(w, Ts, seed, budgets)
    run = G.GpuRun(ctx, K, V, Q, sc, B, w.Hq)
    run.run_all()
    return G.check_against_oracle(run, K, V, Q, sc, B, what)


def test_config0_full(ctx):
    w = W.CONFIGS[0]
    ws, wd = _run_and_check(ctx, w, [4096], what="cfg0")
    print(f"cfg0 worst score ratio {ws:.3g}, worst decode ratio {wd:.3g}")


def test_ragged_small_with_degenerate_budgets(ctx):
    # T not a multiple of any tile; budgets 0, 1, T and in between; GQA group 2
    w = W.scaled(W.CONFIGS[0], L=2, H=3, Hq=6, T=777)
    budgets = [np.array([[0, 1, 777], [300, 64, 5]], dtype=np.int32)]
    _run_and_check(ctx, w, [777], budgets=budgets, what="ragged")


@pytest.mark.parametrize("T", [1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1023, 1025])
def test_tile_boundaries(ctx, T):
    w = W.scaled(W.CONFIGS[0], L=1, H=2, Hq=8, T=T)
    budgets = [np.array([[max(1, T // 3), T - (T > 1)]], dtype=np.int32)]
    _run_and_check(ctx, w, [T], seed=T, budgets=budgets, what=f"T={T}")


def test_several_sequences_of_different_length(ctx):
    w = W.scaled(W.CONFIGS[3], L=2, H=4, Hq=16, n_seq=3, b_min=8)
    _run_and_check(ctx, w, [100, 1000, 5000], what="multi-seq")


@pytest.mark.parametrize("scorer,hidden", [("linear", 0), ("mlp", 32)])
def test_more_sequences_than_one_launch_table_holds(ctx, scorer, hidden):
    # a launch table describes up to 32 sequences: 70 of them take three launches of every kernel
    rng = np.random.default_rng(70)
    Ts = [int(t) for t in rng.integers(20, 400, size=70)]
    Ts[5], Ts[40] = 5000, 17            # mixed tile sizes of the MLP scorer inside one call
    w = W.scaled(W.CONFIGS[0], n_seq=70, L=1, H=2, Hq=4, scorer=scorer, hidden=hidden, act="gelu", b_min=2)
    _run_and_check(ctx, w, Ts, seed=4, what="70 sequences")


@pytest.mark.parametrize("g", [1, 2, 3, 4, 5, 6, 7, 8])
def test_gqa_group_sizes(ctx, g):
    w = W.scaled(W.CONFIGS[0], L=1, H=2, Hq=2 * g, T=1500, b_min=16)
    _run_and_check(ctx, w, [1500], seed=g, what=f"g={g}")


@pytest.mark.parametrize("hidden,act,per_head", [(64, "gelu", False), (32, "silu", True), (16, "gelu", True), (48, "silu", False),
                                                 (128, "silu", True), (80, "gelu", False), (96, "silu", False), (112, "gelu", True),
                                                 (128, "gelu", False)])
def test_mlp_scorer(ctx, hidden, act, per_head):
    w = W.scaled(W.CONFIGS[2], L=2, H=2, Hq=8, T=3000, b_min=16, hidden=hidden, act=act, per_head=per_head)
    ws, wd = _run_and_check(ctx, w, [3000], what=f"mlp{hidden}{act}")
    print(f"mlp {hidden} {act}: worst score ratio {ws:.3g}")


@pytest.mark.parametrize("L,H,hidden,T", [(16, 32, 64, 300), (16, 32, 128, 600), (16, 32, 64, 257), (19, 27, 32, 300), (1, 8, 64, 16385)])
def test_mlp_tiles_that_fill_one_round_of_blocks(ctx, L, H, hidden, T):
    """A launch over one sequence divides the heads evenly over the blocks the chip holds: tiles of 320 rows (the last
    one short), one or more to a head, and a launch over one head too many for that."""
    w = W.scaled(W.CONFIGS[2], L=L, H=H, Hq=H, T=T, b_min=4, hidden=hidden, act="gelu")
    _run_and_check(ctx, w, [T], seed=9, what=f"one round {L}x{H} {hidden} {T}")


@pytest.mark.parametrize("L,H,hidden,Ts", [(1, 8, 64, [9001, 3000, 17]),        # one tile size for all: 448 rows
                                           (1, 8, 64, [40960]), (1, 8, 64, [40961]),   # the most of a block to itself, one more
                                           (1, 8, 128, [12288]), (1, 8, 128, [12289]),
                                           (1, 4, 128, [30001, 257]),             # the two-wave blocks, one round
                                           (16, 32, 64, [1300, 700, 300])])       # several rounds
def test_mlp_tiles_over_all_sequences(ctx, L, H, hidden, Ts):
    w = W.scaled(W.CONFIGS[3], L=L, H=H, Hq=H, T=max(Ts), hidden=hidden, act="silu", per_head=False, b_min=1)
    budgets = [[max(1, T // 40)] * (L * H) for T in Ts]
    _run_and_check(ctx, w, Ts, seed=17, budgets=budgets, what=f"{L} x {H} heads of {Ts}, hidden width {hidden}")


@pytest.mark.parametrize("L,H,hidden,Ts", [(24, 12, 64, [1100]), (24, 12, 128, [900, 900]),   # heads that do not divide a round
                                           (16, 32, 96, [1300]), (16, 32, 32, [1300, 700]),      # narrow: at most 1024 rows
                                           (1, 5, 64, [1500 - 40 * s for s in range(35)])])      # two launches, each its own tiles
def test_mlp_tiles_of_several_rounds(ctx, L, H, hidden, Ts):
    w = W.scaled(W.CONFIGS[3], L=L, H=H, Hq=H, T=max(Ts), hidden=hidden, act="gelu", per_head=False, b_min=1)
    budgets = [[max(1, T // 40)] * (L * H) for T in Ts]
    _run_and_check(ctx, w, Ts, seed=18, budgets=budgets, what=f"{L} x {H} heads of {Ts[:3]}, hidden width {hidden}")


def test_mlp_without_output_bias_and_heavy_tails(ctx):
    w = W.scaled(W.CONFIGS[4], L=2, H=2, Hq=14, T=2500, n_seq=2, b_min=8)
    K, V, Q, sc, B = _inputs(w, [2500, 2500])
    sc["b2"] = None
    run = G.GpuRun(ctx, K, V, Q, sc, B, w.Hq)
    run.run_all()
    G.check_against_oracle(run, K, V, Q, sc, B, "cfg4-like")


def test_paper_scorer_shape(ctx):
    # Sec. 3.4 / Table 5: one 256 -> 128 -> 1 SiLU network per (layer, head), hidden bias, no output bias
    w = W.scaled(W.CONFIGS[5], L=2, H=3, Hq=12, T=2100, b_min=16)
    K, V, Q, sc, B = _inputs(w, [2100])
    assert sc["b2"] is None and sc["w1"].shape == (2, 3, 128, 256)
    run = G.GpuRun(ctx, K, V, Q, sc, B, w.Hq)
    run.run_all()
    G.check_against_oracle(run, K, V, Q, sc, B, "paper scorer")


def test_paper_scorer_count_of_the_deeper_model(ctx):
    # App. C.1: the 36-layer model has 36 x 8 = 288 independent scorers; all of them are exercised here
    w = W.scaled(W.CONFIGS[5], L=36, H=8, Hq=32, T=200, b_min=4)
    K, V, Q, sc, B = _inputs(w, [200])
    assert sc["w1"].shape == (36, 8, 128, 256)
    run = G.GpuRun(ctx, K, V, Q, sc, B, w.Hq)
    run.run_all()
    G.check_against_oracle(run, K, V, Q, sc, B, "288 scorers")


def test_per_head_linear_scorer(ctx):
    w = W.scaled(W.CONFIGS[1], L=3, H=4, Hq=16, T=2048, b_min=8, per_head=True)
    _run_and_check(ctx, w, [2048], what="per-head linear")


@pytest.mark.parametrize("seed", range(24))
def test_random_shapes(ctx, seed):
    # shapes, scorer kinds and budgets drawn at random: several sequences, empty and full heads,
    # lengths off every tile size, GQA groups up to 16
    rng = np.random.default_rng(1000 + seed)
    L, H = int(rng.integers(1, 4)), int(rng.integers(1, 5))
    g = int(rng.choice([1, 2, 3, 4, 5, 7, 8, 12, 16]))
    n_seq = int(rng.integers(1, 4))
    Ts = [int(rng.integers(1, 2600)) for _ in range(n_seq)]
    kind = str(rng.choice(["linear", "mlp"]))
    w = W.scaled(W.CONFIGS[0], L=L, H=H, Hq=H * g, n_seq=n_seq, scorer=kind,
                 hidden=int(rng.choice([16, 32, 64, 80, 128])) if kind == "mlp" else 0,
                 act=str(rng.choice(["silu", "gelu"])), per_head=bool(rng.integers(0, 2)),
                 out_bias=bool(rng.integers(0, 2)))
    budgets = []
    for T in Ts:
        b = rng.integers(0, T + 1, size=(L, H))
        b[rng.random((L, H)) < 0.15] = 0
        b[rng.random((L, H)) < 0.1] = T
        budgets.append(b.astype(np.int32))
    _run_and_check(ctx, w, Ts, seed=seed, budgets=budgets, what=f"random {seed}")


@pytest.mark.parametrize("L,H,Hq,T", [(1, 1, 4, 300), (8, 8, 8, 300), (13, 5, 10, 300), (1, 8, 32, 40000)])
def test_decode_chunks_that_start_at_the_segments_and_flat_ones(ctx, L, H, Hq, T):
    """Up to 64 segments each start their own chunks, more are cut without regard to them.  Segment lengths on either
    side of a tile of 32 rows, of a piece for one wave (64) and of a chunk (128 rows, or 192 for the long heads), and
    empty ones in between."""
    w = W.scaled(W.CONFIGS[0], L=L, H=H, Hq=Hq, T=T, b_min=0)
    edges = [0, 1, 31, 32, 33, 64, 65, 127, 128, 129, 0, 256, 257, T] if T < 1000 else [T, 0, 191, 192, 193, 12345, 1, T - 1]
    budgets = [np.resize(np.array(edges[::-1] if L == 1 and H == 1 else edges, dtype=np.int32), (L, H))]
    _run_and_check(ctx, w, [T], seed=3, budgets=budgets, what=f"decode chunks {L}x{H}")


@pytest.mark.parametrize("lengths,G_", [([1, 33, 64, 65, 700, 0, 2000, 5], 4), ([300] * 64, 1), ([9000], 16)])
def test_decode_over_few_segments_keeps_more_digits_of_the_probabilities(ctx, lengths, G_):
    """Up to 64 segments the probabilities are multiplied in two bf16 parts, relative error 2^-18 each.  An output is a
    weighted mean of value rows, so its error stays below the probabilities' times the largest value; fp32 logits of up
    to 2^4 and exponentials add about 2^-19.  Four times that is allowed (one part alone: 2^-9)."""
    n, total = len(lengths), sum(lengths)
    g = torch.Generator(device="cuda").manual_seed(total)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    q, k, v = normal(1, 1, n * G_, 128), normal(total, 128), normal(total, 128)
    offsets = torch.empty(n + 1, dtype=torch.int32, device="cuda")
    assert lkv.lkv_plan_offsets(ctx, np.array(lengths, dtype=np.int32), offsets) == total
    out = torch.empty(1, 1, n * G_, 128, device="cuda")
    ws = torch.empty(lkv.lkv_decode_workspace_bytes(n, total, n * G_, n), dtype=torch.uint8, device="cuda")
    lkv.lkv_decode_attn(ctx, 1, 1, n, n * G_, 128, q, k, v, offsets, total, 128 ** -0.5, out, None, ws)
    qd, kd, vd, at = q.cpu().double().view(n, G_, 128), k.cpu().double(), v.cpu().double(), 0
    for s, m in enumerate(lengths):
        p = torch.softmax(qd[s] @ kd[at:at + m].T * 128 ** -0.5, dim=1)
        err = (out[0, 0, s * G_:(s + 1) * G_].cpu().double() - p @ vd[at:at + m]).abs().max()
        assert err <= 2.0 ** -16 * vd.abs().max(), (s, m, float(err))
        at += m


@pytest.mark.parametrize("lengths,G_", [([128 * 9, 0, 128 * 64 + 1, 1, 128 * 8, 700], 4),   # parts without a chunk; an empty segment
                                        ([383] * 3, 16), ([384] * 3, 3),                     # either side of three chunks a segment
                                        ([70000], 1), ([100] * 40 + [40000], 8),             # longer chunks; one long among many short
                                        ([128 * 8, 128 * 8 + 1, 0, 128 * 40, 5] * 8, 7),     # more than 256 heads: four threads
                                        ([128 * 8 + 1, 128 * 33] * 32, 16), ([1024, 128] * 16, 8)])
def test_decode_merges_of_many_chunks(ctx, lengths, G_):
    """Segments of up to several hundred chunks, merged by eight or four threads per element.  Errors as in the test above; the log-sum-exp
    is an fp32 sum of fp32 exponentials of logits below 2^4."""
    n, total = len(lengths), sum(lengths)
    g = torch.Generator(device="cuda").manual_seed(total)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    q, k, v = normal(1, 1, n * G_, 128), normal(total, 128), normal(total, 128)
    k[total // 2:] *= 2    # the maxima of the parts differ
    offsets = torch.empty(n + 1, dtype=torch.int32, device="cuda")
    assert lkv.lkv_plan_offsets(ctx, np.array(lengths, dtype=np.int32), offsets) == total
    out = torch.full((1, 1, n * G_, 128), float("nan"), device="cuda")
    lse = torch.full((1, 1, n * G_), float("nan"), device="cuda")
    ws = torch.full((lkv.lkv_decode_workspace_bytes(n, total, n * G_, n),), 255, dtype=torch.uint8, device="cuda")
    lkv.lkv_decode_attn(ctx, 1, 1, n, n * G_, 128, q, k, v, offsets, total, 128 ** -0.5, out, lse, ws)
    qd, kd, vd, at = q.cpu().double().view(n, G_, 128), k.cpu().double(), v.cpu().double(), 0
    for s, m in enumerate(lengths):
        got, got_lse = out[0, 0, s * G_:(s + 1) * G_].cpu().double(), lse[0, 0, s * G_:(s + 1) * G_].cpu().double()
        if m == 0:
            assert (got == 0).all() and torch.isneginf(got_lse).all()
            continue
        x = qd[s] @ kd[at:at + m].T * 128 ** -0.5
        err = (got - torch.softmax(x, dim=1) @ vd[at:at + m]).abs().max()
        assert err <= 2.0 ** -16 * vd.abs().max(), (s, m, float(err))
        assert (got_lse - torch.logsumexp(x, dim=1)).abs().max() <= 2.0 ** -16, (s, m)
        at += m


def test_group_size_limit(ctx):
    w = W.scaled(W.CONFIGS[0], L=1, H=1, Hq=17, T=64, b_min=4)
    K, V, Q, sc, B = _inputs(w, [64])
    run = G.GpuRun(ctx, K, V, Q, sc, B, 16)
    with pytest.raises(lkv.LkvError) as e:
        lkv.lkv_decode_attn(ctx, 1, 1, 1, 17, 128, run.q, run.kp, run.vp, run.offsets, run.total, G.SCALE,
                            run.out, run.lse, run.ws)
    assert e.value.status == 2


def test_all_scores_equal_keeps_the_first_tokens(ctx):
    w = W.scaled(W.CONFIGS[0], L=1, H=2, Hq=8, T=5000)
    K, V, Q, sc, B = _inputs(w, [5000])
    sc["w1"][:] = 0
    run = G.GpuRun(ctx, K, V, Q, sc, B, w.Hq)
    run.run_all()
    idx = run.idx.cpu().numpy()
    off = run.offsets.cpu().numpy()
    for s in range(2):
        assert np.array_equal(idx[off[s]:off[s + 1]], np.arange(off[s + 1] - off[s]))
    G.check_against_oracle(run, K, V, Q, sc, B, "ties")


@pytest.mark.parametrize("T", [12, 63, 4000, 4001, 16383, 16384, 32768, 34304, 34305, 40000, 40003, 131072, 327680, 327681])
def test_select_on_crafted_scores(ctx, T):
    # NaN, infinities, signed zeros, duplicates, values one ulp apart; head lengths on both sides of
    # every storage mode of the kernels (registers, LDS bitmaps, streaming) and off the 16-byte grid
    rng = np.random.default_rng(T)
    H = 4
    k = torch.empty((1, H, T, 128), dtype=torch.bfloat16, device="cuda")   # contents unused by lkv_select
    cache = lkv.Cache([k], [k], H)
    u = rng.standard_normal((1, H, T)).astype(np.float32)
    u[0, 0, ::7] = np.nan; u[0, 0, 5] = -np.inf; u[0, 0, 11] = np.inf
    u[0, 1] = np.round(u[0, 1] * 4) / 4                      # heavy ties
    u[0, 1, ::2] *= 0.0                                      # +0.0 and -0.0
    u[0, 2] = 1.0; u[0, 2, T // 2:] = 1.0 + 2 ** -23          # two values one ulp apart
    u[0, 3] = 0.5                                            # all equal
    budgets = np.minimum(np.array([[T - T // 7 + 3, T // 2, T // 2 + 10, T // 3]], dtype=np.int32), T)
    scores = [torch.from_numpy(u).cuda()]
    total = int(budgets.sum())
    # the index buffer sits inside a larger one so that a kernel writing past its end is caught, not harmful
    buf = torch.full((total + 4 * T + 64,), -1, dtype=torch.int32, device="cuda")
    idx = buf[:total]
    offsets = torch.full((H + 1,), -1, dtype=torch.int32, device="cuda")
    lkv.lkv_select(ctx, cache, scores, budgets, idx, offsets)
    torch.cuda.synchronize()
    idx_ref, off_ref = O.select_all(u, budgets)
    assert np.array_equal(offsets.cpu().numpy(), off_ref)
    assert bool((buf[total:] == -1).all()), "writes past the end of idx"
    got = idx.cpu().numpy()
    for h in range(H):
        assert np.array_equal(got[off_ref[h]:off_ref[h + 1]], idx_ref[off_ref[h]:off_ref[h + 1]]), f"head {h}"


@pytest.mark.parametrize("lengths", [(8192, 8193), (16384, 16385), (34816, 34817), (1023, 40001, 513, 34816)])
@pytest.mark.parametrize("budget_share", [0.003, 0.15, 0.9])
def test_select_on_distributions_the_bins_do_not_spread(ctx, lengths, budget_share):
    # Either side of every kernel size, and short and long sequences in one call.  Distributions: plain; one value far from
    # the rest (all others share a bin); +inf on a stretch, as a window scorer leaves it; a narrow cluster at the threshold
    # (more than can be ranked one by one, and more than the list of a long head holds); ties at the threshold; values
    # whose squares overflow.  Exact, so against the oracle's sort.
    H = 6
    rng = np.random.default_rng(sum(lengths))
    us = []
    for T in lengths:
        u = rng.standard_normal((1, H, T)).astype(np.float32)
        u[0, 1, T // 3] = 1e30
        u[0, 2, T - min(T // 4, 100):] = np.inf
        n_top = max(1, int(T * budget_share) - 700)
        u[0, 3] = 1.0 + rng.integers(0, 64, T).astype(np.float32) * np.float32(2 ** -23)
        u[0, 3, rng.permutation(T)[:n_top]] = 2.0
        u[0, 4] = np.round(u[0, 4] * 8) / 8
        u[0, 5] *= np.float32(1e30)
        u[0, 5, ::11] = np.nan
        us.append(u)
    kv = [torch.empty((1, H, T, 128), dtype=torch.bfloat16, device="cuda") for T in lengths]   # contents unused by lkv_select
    cache = lkv.Cache(kv, kv, H)
    budgets = np.concatenate([np.full(H, max(1, int(T * budget_share)), dtype=np.int32) + np.arange(H, dtype=np.int32) for T in lengths])
    scores = [torch.from_numpy(u).cuda() for u in us]
    total = int(budgets.sum())
    idx = torch.full((total + 64,), -1, dtype=torch.int32, device="cuda")
    offsets = torch.empty(budgets.size + 1, dtype=torch.int32, device="cuda")
    counts = torch.empty(lkv.lkv_counts_bytes(budgets.size), dtype=torch.uint8, device="cuda")
    ref = [O.select(us[s // H][0, s % H], int(b)) for s, b in enumerate(budgets)]
    for counted in (False, True):
        idx.fill_(-1)
        if counted:   # the first-level digits as a scoring launch leaves them
            keys = [np.where(np.isnan(u), -np.inf, u).astype(np.float32).view(np.uint32) for u in us]
            keys = [np.where(k >> 31, ~k, k | np.uint32(0x80000000)) >> 21 for k in keys]
            hist = np.stack([np.bincount(k[0, h], minlength=2048) for k in keys for h in range(H)]).astype(np.int32)
            counts[:] = torch.from_numpy(hist.reshape(-1).view(np.uint8)).cuda()
            lkv.lkv_select_counted(ctx, cache, scores, budgets, counts, idx, offsets)
        else:
            lkv.lkv_select(ctx, cache, scores, budgets, idx, offsets)
        torch.cuda.synchronize()
        got, off = idx.cpu().numpy(), offsets.cpu().numpy()
        assert (got[total:] == -1).all(), "writes past the end of idx"
        for s, r in enumerate(ref):
            assert np.array_equal(got[off[s]:off[s + 1]], r), (counted, "sequence", s // H, "head", s % H)
        if counted:
            assert not bool(counts.any()), "counters left behind"


@pytest.mark.parametrize("n_top", [16383, 16384, 16385, 30000])
def test_select_long_head_candidate_list_limit(ctx, n_top):
    # a head too long for the registers: after the first radix level the undecided bin holds n_top keys;
    # up to 16384 of them are listed in LDS, more fall back to re-reading the scores
    rng = np.random.default_rng(n_top)
    T, H = 50000, 2
    k = torch.empty((1, H, T, 128), dtype=torch.bfloat16, device="cuda")
    cache = lkv.Cache([k], [k], H)
    u = rng.uniform(-6.0, -2.0, size=(1, H, T)).astype(np.float32)
    for h in range(H):
        where = rng.choice(T, size=n_top, replace=False)
        u[0, h, where] = rng.uniform(1.0, 1.18, size=n_top).astype(np.float32)     # one bin of the first level
    u[0, 1, ::3] = np.float32(1.0625)                                              # and many ties inside it
    budgets = np.array([[n_top // 2, n_top // 3 + 7]], dtype=np.int32)
    total = int(budgets.sum())
    buf = torch.full((total + 64,), -1, dtype=torch.int32, device="cuda")
    offsets = torch.full((H + 1,), -1, dtype=torch.int32, device="cuda")
    lkv.lkv_select(ctx, cache, [torch.from_numpy(u).cuda()], budgets, buf[:total], offsets)
    torch.cuda.synchronize()
    idx_ref, off_ref = O.select_all(u, budgets)
    assert bool((buf[total:] == -1).all()), "writes past the end of idx"
    assert np.array_equal(buf[:total].cpu().numpy(), idx_ref)


def test_select_mixed_lengths_in_one_launch(ctx):
    # sequences whose heads use different storage modes share one launch (and one LDS size)
    rng = np.random.default_rng(5)
    Ts = [3000, 50000, 34304, 70001]
    H = 2
    ks = [torch.empty((1, H, T, 128), dtype=torch.bfloat16, device="cuda") for T in Ts]
    cache = lkv.Cache(ks, ks, H)
    us = [rng.standard_normal((1, H, T)).astype(np.float32) for T in Ts]
    budgets = np.array([[T // 5, T // 9] for T in Ts], dtype=np.int32)
    total = int(budgets.sum())
    idx = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    offsets = torch.full((len(Ts) * H + 1,), -1, dtype=torch.int32, device="cuda")
    lkv.lkv_select(ctx, cache, [torch.from_numpy(u).cuda() for u in us], budgets.reshape(-1), idx, offsets)
    torch.cuda.synchronize()
    got = idx.cpu().numpy()
    off = offsets.cpu().numpy()
    assert np.array_equal(off, np.concatenate([[0], np.cumsum(budgets.reshape(-1))]))
    for s, T in enumerate(Ts):
        for h in range(H):
            seg = s * H + h
            assert np.array_equal(got[off[seg]:off[seg + 1]], O.select(us[s][0, h], int(budgets[s, h]))), (s, h)


def test_results_are_reproducible(ctx):
    w = W.scaled(W.CONFIGS[0], L=1, H=4, Hq=16, T=9000)
    K, V, Q, sc, B = _inputs(w, [9000])
    run = G.GpuRun(ctx, K, V, Q, sc, B, w.Hq)
    run.run_all()
    first = (run.idx.clone(), run.kp.clone(), run.out.clone())
    for _ in range(3):
        run.run_all()
        assert torch.equal(run.idx, first[0]) and torch.equal(run.kp, first[1]) and torch.equal(run.out, first[2])


def test_argument_errors_are_reported_before_launch(ctx):
    w = W.scaled(W.CONFIGS[0], L=1, H=2, Hq=8, T=128, b_min=4)
    K, V, Q, sc, B = _inputs(w, [128])
    run = G.GpuRun(ctx, K, V, Q, sc, B, w.Hq)
    bad = run.budgets.copy(); bad[1] = 129
    with pytest.raises(lkv.LkvError) as e:
        lkv.lkv_select(ctx, run.cache, run.scores, bad, run.idx, run.offsets)
    assert e.value.status == 1 and "129" in str(e.value)
    with pytest.raises(lkv.LkvError) as e:
        lkv.lkv_decode_attn(ctx, 1, 1, 2, 8, 128, run.q, run.kp, run.vp, run.offsets, run.total, G.SCALE,
                            run.out, run.lse, None)
    assert e.value.status == 3
    with pytest.raises(lkv.LkvError) as e:
        lkv.lkv_decode_attn(ctx, 1, 1, 2, 8, 64, run.q, run.kp, run.vp, run.offsets, run.total, G.SCALE,
                            run.out, run.lse, run.ws)
    assert e.value.status == 2
    torch.cuda.synchronize()
