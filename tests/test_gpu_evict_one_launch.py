"""Top-k and compaction of a layer view in one launch (lkv_evict_layer, short heads and few of them) against the general
path, lkv_select and lkv_compact over the same scores, bit for bit; and the indices against the oracle's top-k."""
import numpy as np
import pytest
import torch

from oracle import lkv_oracle as O
from paper_2605_06676_amd import lkv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = lkv.Context(0)
    yield c
    c.close()


def draw_scores(kind, shape, rng):
    u = rng.standard_normal(shape).astype(np.float32)
    if kind == "ties":            # few values, each many times: more copies of the threshold than are ranked one by one
        u = np.round(u * 2) / 2
    elif kind == "equal":
        u = np.full(shape, -0.5, np.float32)
    elif kind == "special":
        flat = u.reshape(-1)
        for x in (np.nan, np.inf, -np.inf, 0.0, -0.0, 1e30, -1e30):
            flat[rng.integers(0, flat.size, max(1, flat.size // 50))] = x
    elif kind == "late":          # what is kept lies at the end of the head
        u += np.linspace(0, 20, shape[-1], dtype=np.float32)
    return u


# sequence lengths, layers of the model and of the view, heads, and the kinds of scores
CASES = [
    ([1], 1, 1, 1, "normal"), ([63], 2, 1, 2, "normal"), ([64], 1, 1, 3, "special"), ([65, 1], 3, 2, 2, "normal"),
    ([1023], 1, 1, 2, "ties"), ([1024], 1, 1, 2, "normal"), ([1025, 3000], 2, 1, 4, "special"),
    ([8192], 1, 1, 8, "normal"), ([8193], 1, 1, 8, "late"), ([16384], 1, 1, 2, "equal"), ([16385, 700, 9001], 2, 2, 2, "ties"),
    ([34816], 1, 1, 2, "normal"), ([34816, 17], 3, 2, 1, "special"), ([34000], 2, 2, 4, "late"), ([20001], 1, 1, 3, "ties"),
    ([300], 8, 8, 8, "normal"),                       # 64 heads
    ([300, 40], 11, 11, 3, "normal"),                 # 66: the general path
    ([34817], 1, 1, 2, "normal"), ([34817, 900], 1, 1, 1, "ties"),   # too long for the registers
]


@pytest.mark.parametrize("counted", [False, True])
@pytest.mark.parametrize("lens,n_layers,m,H,kind", CASES)
def test_same_as_select_and_compact(ctx, lens, n_layers, m, H, kind, counted):
    rng = np.random.default_rng(len(lens) * 1000 + lens[0] + H)
    K = [torch.randint(-30000, 30000, (m, H, T, 128), dtype=torch.int16, device="cuda").view(torch.bfloat16) for T in lens]
    V = [torch.randint(-30000, 30000, (m, H, T, 128), dtype=torch.int16, device="cuda").view(torch.bfloat16) for T in lens]
    view = lkv.Cache(K, V, H)
    u = [draw_scores(kind, (m, H, T), rng) for T in lens]
    scores = [torch.from_numpy(x).cuda() for x in u]
    budgets = np.zeros((len(lens), n_layers, H), np.int32)
    layer = n_layers - m
    for s, T in enumerate(lens):
        b = rng.integers(0, T + 1, size=(n_layers, H))
        b[:, 0] = rng.choice([0, 1, T - 1, T, T // 2], n_layers)
        b[layer, -1] = max(1, T // 7)
        budgets[s] = b
    offsets = torch.empty(budgets.size + 1, dtype=torch.int32, device="cuda")
    total = lkv.lkv_plan_offsets(ctx, budgets, offsets)
    idx = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    kp, vp = (torch.zeros((total, 128), dtype=torch.int16, device="cuda").view(torch.bfloat16) for _ in range(2))
    counts = None
    if counted:   # with a NULL scorer nothing counts and the buffer stays as it is
        counts = torch.zeros(lkv.lkv_counts_bytes(budgets.size), dtype=torch.uint8, device="cuda")
    lkv.lkv_evict_layer(ctx, view, layer, n_layers, None, budgets, offsets, scores, idx, kp, vp, counts=counts)

    mine = np.ascontiguousarray(budgets[:, layer:layer + m])
    offsets2 = torch.empty(mine.size + 1, dtype=torch.int32, device="cuda")
    n = lkv.lkv_plan_offsets(ctx, mine, offsets2)
    idx2 = torch.empty(max(n, 1), dtype=torch.int32, device="cuda")
    kp2, vp2 = (torch.empty((max(n, 1), 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    lkv.lkv_select(ctx, view, scores, None, idx2, offsets2)
    lkv.lkv_compact(ctx, view, idx2, offsets2, n, kp2, vp2)
    torch.cuda.synchronize()
    off, off2 = offsets.cpu().numpy(), offsets2.cpu().numpy()
    touched = np.zeros(total, bool)
    for s, T in enumerate(lens):
        for j in range(m * H):
            a = (s * n_layers + layer) * H + j
            lo, hi, l2, h2 = off[a], off[a + 1], off2[s * m * H + j], off2[s * m * H + j + 1]
            assert hi - lo == h2 - l2
            touched[lo:hi] = True
            assert torch.equal(idx[lo:hi], idx2[l2:h2]), (s, j)
            assert np.array_equal(idx[lo:hi].cpu().numpy(), O.select(u[s].reshape(m * H, T)[j], int(hi - lo))), (s, j)
            assert torch.equal(kp[lo:hi].view(torch.int16), kp2[l2:h2].view(torch.int16))
            assert torch.equal(vp[lo:hi].view(torch.int16), vp2[l2:h2].view(torch.int16))
    # rows of other layers are not written
    rest = torch.from_numpy(~touched).cuda()
    assert (idx[rest] == -1).all() and (kp[rest].view(torch.int16) == 0).all() and (vp[rest].view(torch.int16) == 0).all()


def test_counters_are_left_zero(ctx):
    # the scoring launch counts, the one launch of short heads does not need the counts and clears them
    g = torch.Generator(device="cuda").manual_seed(3)
    k, v = (torch.randn((2, 3, 5000, 128), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    view = lkv.Cache([k], [v], 3)
    w1 = torch.randn((2, 32, 256), device="cuda", generator=g).mul(0.05).to(torch.bfloat16)
    scorer = {"kind": "mlp", "act": "silu", "hidden": 32, "per_head": False, "w1": w1, "w2": torch.randn((2, 32), device="cuda", generator=g),
              "b1": torch.zeros((2, 32), device="cuda"), "b2": None}
    budgets = np.array([0, 700, 5000, 1, 4999, 333], np.int32)
    offsets = torch.empty(7, dtype=torch.int32, device="cuda")
    total = lkv.lkv_plan_offsets(ctx, budgets, offsets)
    idx = torch.empty(total, dtype=torch.int32, device="cuda")
    kp, vp = (torch.empty((total, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    counts = torch.zeros(lkv.lkv_counts_bytes(6), dtype=torch.uint8, device="cuda")
    u = torch.empty((2, 3, 5000), device="cuda")
    for _ in range(3):
        lkv.lkv_evict_layer(ctx, view, 0, 2, scorer, budgets, offsets, [u], idx, kp, vp, counts=counts)
    torch.cuda.synchronize()
    assert not counts.any()
    uh, off = u.cpu().numpy().reshape(6, 5000), offsets.cpu().numpy()
    for j in range(6):
        assert np.array_equal(idx[off[j]:off[j + 1]].cpu().numpy(), O.select(uh[j], int(budgets[j])))


# longer heads: classified by several blocks with the counts of the scoring launch, settled in every block that copies
LONG = [([34817], 1, 1, 2), ([40000], 2, 1, 8), ([65537, 34900], 1, 1, 2), ([131077], 1, 1, 1), ([327680], 1, 1, 1),
        ([36001], 4, 4, 4), ([36001], 5, 5, 4),         # 16 heads, 20 (two launches)
        ([327681], 1, 1, 1), ([50000, 20000], 1, 1, 1)]  # too long for the bitmaps; one too short to be split


@pytest.mark.parametrize("kind", ["plain", "narrow", "steps", "equal"])
@pytest.mark.parametrize("lens,n_layers,m,H", LONG)
def test_long_heads_same_as_select_and_compact(ctx, lens, n_layers, m, H, kind):
    rng = np.random.default_rng(lens[0] + H)
    g = torch.Generator(device="cuda").manual_seed(lens[0])
    K, V = ([torch.empty((m, H, T, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for T in lens] for _ in range(2))
    view = lkv.Cache(K, V, H)
    w2 = torch.randn((n_layers, 16), device="cuda", generator=g)
    scorer = {"kind": "mlp", "act": "silu", "hidden": 16, "per_head": False, "b1": torch.zeros((n_layers, 16), device="cuda"), "w2": w2, "b2": None,
              "w1": torch.randn((n_layers, 16, 256), device="cuda", generator=g).mul(0.05).to(torch.bfloat16)}
    if kind == "narrow":      # one first digit for all: more than can be listed
        scorer["b2"] = torch.full((n_layers,), 1000.0, device="cuda")
    elif kind == "steps":     # few values, many copies of the threshold
        scorer["b2"] = torch.full((n_layers,), 3e5, device="cuda")
    elif kind == "equal":
        scorer["w2"] = w2 * 0
    budgets = np.zeros((len(lens), n_layers, H), np.int32)
    for s, T in enumerate(lens):
        budgets[s] = rng.integers(1, T // 5, size=(n_layers, H))
        if H > 1:
            budgets[s, :, 0] = rng.choice([0, 1, 300, T // 2], n_layers)
    if len(lens) == 1 and H == 1:
        budgets[0, :, 0] = lens[0] // 3
    offsets = torch.empty(budgets.size + 1, dtype=torch.int32, device="cuda")
    total = lkv.lkv_plan_offsets(ctx, budgets, offsets)
    idx = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    kp, vp = (torch.zeros((total, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    counts = torch.zeros(lkv.lkv_counts_bytes_split(budgets.size, max(lens)), dtype=torch.uint8, device="cuda")
    scores = [torch.empty((m, H, T), device="cuda") for T in lens]
    layer = n_layers - m
    for _ in range(2):        # the second call finds the counters as the first one left them
        lkv.lkv_evict_layer(ctx, view, layer, n_layers, scorer, budgets, offsets, scores, idx, kp, vp, counts=counts)
    mine = np.ascontiguousarray(budgets[:, layer:layer + m])
    offsets2 = torch.empty(mine.size + 1, dtype=torch.int32, device="cuda")
    n = lkv.lkv_plan_offsets(ctx, mine, offsets2)
    idx2 = torch.empty(max(n, 1), dtype=torch.int32, device="cuda")
    kp2, vp2 = (torch.empty((max(n, 1), 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    lkv.lkv_select(ctx, view, scores, None, idx2, offsets2)
    lkv.lkv_compact(ctx, view, idx2, offsets2, n, kp2, vp2)
    torch.cuda.synchronize()
    assert not counts[:lkv.lkv_counts_bytes(budgets.size)].any()
    off, off2 = offsets.cpu().numpy(), offsets2.cpu().numpy()
    for s, T in enumerate(lens):
        for j in range(m * H):
            a = (s * n_layers + layer) * H + j
            lo, hi, l2, h2 = off[a], off[a + 1], off2[s * m * H + j], off2[s * m * H + j + 1]
            assert torch.equal(idx[lo:hi], idx2[l2:h2]), (s, j)
            assert torch.equal(kp[lo:hi].view(torch.int16), kp2[l2:h2].view(torch.int16))
            assert torch.equal(vp[lo:hi].view(torch.int16), vp2[l2:h2].view(torch.int16))


@pytest.mark.parametrize("dirt", ["ones", "many", "negative", "low", "random"])
@pytest.mark.parametrize("T,H", [(34817, 2), (40000, 8), (131077, 1)])
def test_counters_that_are_not_zero_on_entry_lead_out_of_no_head(ctx, T, H, dirt):
    # a caller's error: which rows are kept means nothing then, but they are rows of the head, copied as the index says, the
    # rows of other layers stay as they are, and the counters are zero again for the next call
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V = (torch.empty((1, H, T, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(2))
    view = lkv.Cache([K], [V], H)
    scorer = {"kind": "mlp", "act": "silu", "hidden": 16, "per_head": False, "b1": torch.zeros((2, 16), device="cuda"), "b2": None,
              "w1": torch.randn((2, 16, 256), device="cuda", generator=g).mul(0.05).to(torch.bfloat16),
              "w2": torch.randn((2, 16), device="cuda", generator=g)}
    budgets = np.full((2, H), T // 11, np.int32)
    n_seg = 2 * H
    offsets = torch.empty(n_seg + 1, dtype=torch.int32, device="cuda")
    total = lkv.lkv_plan_offsets(ctx, budgets, offsets)
    idx = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    kp, vp = (torch.zeros((total, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    counts = torch.zeros(lkv.lkv_counts_bytes_split(n_seg, T) // 4, dtype=torch.int32, device="cuda")
    mine = counts[:n_seg * 2048].view(n_seg, 2048)[:H]        # of layer 0
    if dirt == "ones":
        mine += 1
    elif dirt == "many":
        mine[:, 1100:] = T
    elif dirt == "negative":                                   # the bin found lies too low: too many tokens above it
        mine[:, 1024:] = -40
    elif dirt == "low":
        mine[:, :300] = 1 << 30
    else:
        mine.random_(-2 ** 31, 2 ** 31 - 1, generator=g)
    scores = torch.empty((1, H, T), device="cuda")
    lkv.lkv_evict_layer(ctx, view, 0, 2, scorer, budgets, offsets, [scores], idx, kp, vp, counts=counts)
    torch.cuda.synchronize()
    assert not counts[:n_seg * 2048].any()
    b, half = T // 11, total // 2
    got = idx[:half].view(H, b).long()
    assert (got >= 0).all() and (got < T).all()
    for h in range(H):
        assert torch.equal(kp[h * b:(h + 1) * b].view(torch.int16), K[0, h][got[h]].view(torch.int16))
        assert torch.equal(vp[h * b:(h + 1) * b].view(torch.int16), V[0, h][got[h]].view(torch.int16))
    assert (idx[half:] == -1).all() and (kp[half:].view(torch.int16) == 0).all() and (vp[half:].view(torch.int16) == 0).all()
    lkv.lkv_evict_layer(ctx, view, 0, 2, scorer, budgets, offsets, [scores], idx, kp, vp, counts=counts)
    u = scores.cpu().numpy()[0]
    for h in range(H):
        assert np.array_equal(idx[h * b:(h + 1) * b].cpu().numpy(), O.select(u[h], b))


@pytest.mark.parametrize("n_streams", [2, 4])
@pytest.mark.parametrize("T,H,counted", [(5000, 8, False), (20001, 4, True), (34816, 2, False), (40000, 4, True), (65537, 2, True)])
def test_layers_evicted_on_several_streams_at_once(ctx, T, H, counted, n_streams):
    # eight layers, enqueued in turn on the streams without a wait between them, into one packed cache, with one counter buffer:
    # the same as one layer after the other, in every round
    L = 8
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V = ([torch.empty((1, H, T, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(L)] for _ in range(2))
    views = [lkv.Cache([K[l]], [V[l]], H) for l in range(L)]
    scorer = {"kind": "mlp", "act": "silu", "hidden": 16, "per_head": False, "b1": torch.zeros((L, 16), device="cuda"), "b2": None,
              "w1": torch.randn((L, 16, 256), device="cuda", generator=g).mul(0.05).to(torch.bfloat16),
              "w2": torch.randn((L, 16), device="cuda", generator=g)}
    rng = np.random.default_rng(T)
    budgets = rng.integers(0, T // 6, size=(L, H)).astype(np.int32)
    budgets[1, 0], budgets[2, -1] = 0, T // 3
    offsets = torch.empty(L * H + 1, dtype=torch.int32, device="cuda")
    total = lkv.lkv_plan_offsets(ctx, budgets, offsets)
    counts = torch.zeros(lkv.lkv_counts_bytes_split(L * H, T) // 4, dtype=torch.int32, device="cuda") if counted else None
    streams = [torch.cuda.Stream() for _ in range(n_streams)]
    scratch = [torch.empty((1, H, T), device="cuda") for _ in range(n_streams)]

    def evict(on):
        idx = torch.full((total,), -1, dtype=torch.int32, device="cuda")
        kp, vp = (torch.zeros((total, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        for l in range(L):
            j = l % n_streams
            lkv.lkv_evict_layer(ctx, views[l], l, L, scorer, budgets, offsets, [scratch[j]], idx, kp, vp,
                                stream=streams[j] if on else None, counts=counts)
        torch.cuda.synchronize()
        assert counts is None or not counts[:L * H * 2048].any()
        return idx, kp.view(torch.int16), vp.view(torch.int16)

    one_by_one = evict(False)
    off = offsets.cpu().numpy()
    for l in range(0, L, 3):      # and these are the oracle's, on the scores of the general path
        u = torch.empty((1, H, T), device="cuda")
        sl = dict(scorer, w1=scorer["w1"][l:l + 1], b1=scorer["b1"][l:l + 1], w2=scorer["w2"][l:l + 1])
        lkv.lkv_score(ctx, views[l], sl, [u])
        uh = u.cpu().numpy()[0]
        for h in range(H):
            a, b = off[l * H + h], off[l * H + h + 1]
            assert np.array_equal(one_by_one[0][a:b].cpu().numpy(), O.select(uh[h], int(b - a)))
    for _ in range(4):
        for got, want in zip(evict(True), one_by_one):
            assert torch.equal(got, want)
