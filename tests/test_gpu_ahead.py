"""talon_build_tree with rows scanned ahead of the tree (talon_build_tree_ahead) against the loop that
scans one layer after the other, and against torch where the row order is adversarial."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def rows_of(B, N, V, dtype, seed, lo=0.5, hi=4.0):
    import torch
    on = "cuda" if B * N * V > 5e7 else "cpu"
    g = torch.Generator(device=on).manual_seed(seed)
    x = torch.randn(B, N, V, generator=g, device=on) * (lo + (hi - lo) * torch.rand(B, N, 1, generator=g, device=on))
    V8 = (V + 7) // 8 * 8
    pool = torch.zeros(B, N, V8, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device=on)
    pool[:, :, :V] = x.to(pool.dtype)
    return pool.cuda()[:, :, :V]


def build(logits, N, k, Dmax, ahead, K_init=None, init_layers=1, mu=0.03):
    """One tree per sequence; candidate arrays start from a sentinel."""
    import torch
    import paper_2601_07353_amd as T
    B, _, V = logits.shape
    st = T.TreeState(B, N)
    cand = T.Candidates(B, st.N_pad, k)
    for t in (cand.token, cand.logit, cand.prob, cand.edge_logp, cand.row_max, cand.row_lse):
        t.fill_(-77)
    dt = T.TALON_DTYPE_F32 if logits.dtype == torch.float32 else T.TALON_DTYPE_BF16
    ws = T.make_expand_workspace(B, st.N_pad, V, k, dt)
    roots = torch.arange(B, dtype=torch.int32).cuda()
    mask = torch.full((B, st.N_pad, st.N_pad // 64), -1, dtype=torch.int64, device="cuda")
    for _ in range(2):   # the second call finds the workspace as the first one left it
        if ahead:
            T.talon_build_tree(roots, logits, st, k, mu, K_init or k, init_layers, Dmax, cand, ws, mask=mask)
        else:
            T.talon_tree_init(st, roots)
            T.talon_expand_tree(logits, st, k, mu, K_init or k, init_layers, Dmax, cand, ws)
            T.talon_build_tree_mask(st, mask)
    torch.cuda.synchronize()
    out = {n: getattr(st, n).cpu().numpy() for n in ("token", "parent", "depth", "prob", "logp", "n_nodes", "frontier_begin",
                                                     "frontier_count", "depth_cur", "status")}
    out["mask"] = mask.cpu().numpy()
    out.update({"cand_" + n: getattr(cand, n).cpu().numpy() for n in ("token", "logit", "prob", "edge_logp", "row_max", "row_lse")})
    return out


def same(a, b):
    for key in a:
        if key in ("prob", "logp", "cand_prob", "cand_edge_logp", "cand_row_lse"):
            # sums of a row's chunks in another order: 2e-6 on a log-sum-exp, one per layer of a path
            np.testing.assert_allclose(a[key], b[key], rtol=1e-5, atol=2e-6 * 24, err_msg=key)
        else:
            np.testing.assert_array_equal(a[key], b[key], err_msg=key)


@pytest.mark.parametrize("B,V,dtype,k,N,Dmax,init_layers", [
    (1, 8, "f32", 2, 2, 4, 1),            # two nodes: one row
    (2, 5, "bf16", 8, 17, 6, 1),          # fewer tokens than candidates
    (3, 5003, "bf16", 31, 130, 12, 1),    # more than 128 frontier rows with the most candidates a row may have then
    (2, 3001, "f32", 64, 64, 8, 1),       # the largest cap
    (1, 70001, "f32", 4, 255, 24, 0),     # many short runs per row, no top-K layer
    (70, 1025, "bf16", 4, 20, 5, 1),      # more sequences than a wavefront has lanes
    (8, 20000, "bf16", 16, 256, 24, 2),   # 2040 rows: scanners take further items from the counter
    (2, 8192, "bf16", 10, 60, 1, 1),      # one layer: scanned layer by layer
    (16, 151936, "bf16", 16, 60, 12, 1),  # a budget near the first layer's width: scanned layer by layer
    (3, 128256, "bf16", 8, 200, 2, 1),    # two layers: 9 rows of 199 are scanned
    (2, 20000, "f32", 8, 128, 3, 0),      # three layers: 73 rows of 127
    (8, 128256, "f32", 16, 256, 24, 1),   # several runs per row, shorter ones for the first rows
])
def test_rows_scanned_ahead_build_the_same_trees(B, V, dtype, k, N, Dmax, init_layers):
    logits = rows_of(B, N, V, dtype, seed=100 * N + k)
    same(build(logits, N, k, Dmax, True, init_layers=init_layers), build(logits, N, k, Dmax, False, init_layers=init_layers))


@pytest.mark.parametrize("spare", [-1, 0, 1, -20])
def test_rows_the_tree_does_not_need_have_no_effect(spare):
    """N-1 rows are the most a tree expands.  The rows no node of this tree expands hold NaN; with
    fewer rows than N-1 the call scans layer by layer and never touches what is not there."""
    import torch
    N, k = 60, 10
    logits = rows_of(1, N, 30000, "bf16", seed=5)
    want = build(logits, N, k, 12, False)
    expanded = int(want["frontier_begin"][0])
    rows = max(N + spare, expanded)
    cut = logits[:, :rows].clone()
    cut[:, expanded:] = float("nan")
    got = build(cut, N, k, 12, True)
    same(got, want)
    assert got["status"][0] == 1


def test_a_bad_row_stops_its_sequence_only():
    import paper_2601_07353_amd as T
    logits = rows_of(3, 40, 9000, "f32", seed=9)
    logits[1, 3, 77] = float("nan")
    a, b = build(logits, 40, 8, 8, True), build(logits, 40, 8, 8, False)
    assert a["status"].tolist() == b["status"].tolist() and a["status"][1] == T.binding.TALON_STATUS_BAD_ROW
    for key in ("token", "parent", "n_nodes", "depth_cur", "frontier_begin", "frontier_count", "mask"):
        np.testing.assert_array_equal(a[key], b[key], err_msg=key)


@pytest.mark.parametrize("B", [1, 66])
def test_forms_take_turns_on_a_workspace_in_mid_tree(B):
    """A tree continued from its second layer leaves descriptors whose first word is not zero; the other
    forms must not read them."""
    import torch
    import paper_2601_07353_amd as T
    N, k, Dmax = 40, 6, 8
    logits = rows_of(B, N, 3000, "f32", seed=3)
    want = build(logits, N, k, Dmax, False)
    st = T.TreeState(B, N)
    cand = T.Candidates(B, st.N_pad, k)
    ws = T.make_expand_workspace(B, st.N_pad, 3000, k, T.TALON_DTYPE_F32)
    roots = torch.arange(B, dtype=torch.int32).cuda()

    def check():
        torch.cuda.synchronize()
        for key in ("token", "parent", "n_nodes", "status"):
            np.testing.assert_array_equal(getattr(st, key).cpu().numpy(), want[key], err_msg=key)

    for _ in range(2):
        T.talon_tree_init(st, roots)
        for d in range(2):
            T.talon_expand_select_layer(logits, st, k, 0.03, k, 1, Dmax, cand, ws, layer=d)
        T.talon_expand_tree(logits, st, k, 0.03, k, 1, Dmax, cand, ws)
        check()
        T.talon_build_tree(roots, logits, st, k, 0.03, k, 1, Dmax, cand, ws)
        check()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("order", ["ascending", "descending", "sawtooth", "ascending late"])
def test_scan_of_rows_in_adversarial_order(dtype, order):
    """Rows that rise along the token ids raise the scan's threshold group by group; the k best and
    the log-sum-exp must not notice."""
    import torch
    V, k = 41003, 16
    x = torch.arange(V, dtype=torch.float32) * (20.0 / V)
    if order == "descending":
        x = x.flip(0)
    elif order == "sawtooth":
        x = (torch.arange(V) * 2049 % V).float() * (20.0 / V)
    elif order == "ascending late":
        x[: V // 2] = 0.0
    logits = torch.zeros(1, 12, (V + 7) // 8 * 8, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    logits[:, :, :V] = x.to(logits.dtype)
    logits = logits.cuda()[:, :, :V]
    got = build(logits, 12, k, 4, True)
    row = logits[0, 0].double().cpu()
    order_ids = torch.argsort(row, descending=True, stable=True)[:k]     # equal logits: lower token first
    np.testing.assert_array_equal(got["cand_token"][0, 0], order_ids.numpy())
    assert abs(got["cand_row_lse"][0, 0] - float(torch.logsumexp(row, 0))) < 2e-6


@pytest.mark.parametrize("B", [1, 2, 65, 150])
def test_one_launch_per_layer_with_bad_rows_and_finished_sequences(B):
    """A launch per layer takes the status of a sequence from the launch's start and counts the selections
    that have seen the whole grid start: more sequences than a wavefront has lanes, rows that cannot be
    normalised (in the first layer and in later ones), sequences that end early; twice over one
    workspace.  Reference: the separate calls, with the same trees to the last bit (same chunks of one)."""
    import torch
    import paper_2601_07353_amd as T
    V, N, k, Dmax = 700, 12, 3, 5
    logits = rows_of(B, N, V, "f32", seed=11).clone()
    logits[::7, 0, 5] = float("nan")        # no first layer
    logits[1::5, 2, 9] = float("inf")       # none below node 2, where a tree has one
    logits[B - 1, 0, 3] = 80.0              # a sure row
    st = T.TreeState(B, N)
    cand = T.Candidates(B, st.N_pad, k)
    ws = T.make_expand_workspace(B, st.N_pad, V, k, T.TALON_DTYPE_F32)
    roots = torch.arange(B, dtype=torch.int32).cuda()
    fields = ("token", "parent", "depth", "prob", "logp", "n_nodes", "frontier_begin", "frontier_count", "depth_cur", "status")

    def snapshot():
        torch.cuda.synchronize()
        n = st.n_nodes.cpu()
        return {f: [getattr(st, f)[b, : n[b]].cpu().numpy() if getattr(st, f).dim() == 2 else int(getattr(st, f)[b]) for b in range(B)]
                for f in fields}

    T.talon_tree_init(st, roots)
    for d in range(Dmax):
        T.talon_expand_layer(logits, st, k, cand, ws, layer=d)
        T.talon_select_budget(st, k, cand, 0.03, k, 1, Dmax)
    want = snapshot()
    bad = T.binding.TALON_STATUS_BAD_ROW
    assert want["status"][0] & bad and (B < 3 or not want["status"][2] & bad)
    for _ in range(2):
        T.talon_tree_init(st, roots)
        for d in range(Dmax):
            T.talon_expand_select_layer(logits, st, k, 0.03, k, 1, Dmax, cand, ws, layer=d)
        got = snapshot()
        for f in fields:
            for b in range(B):
                np.testing.assert_array_equal(got[f][b], want[f][b], err_msg="%s of sequence %d" % (f, b))


@pytest.mark.parametrize("rows,k,N,equal", [
    (2, 16, 20, True),       # 32 equal scores, 17 of them fit: the first ones in (parent, rank) order
    (2, 60, 67, True),       # 120 equal scores, 64 places
    (4, 5, 18, False),       # 20 candidates for 13 places
    (8, 16, 109, False),     # 128 for 100: the most that are ranked so
    (3, 43, 90, False),      # 129 for 86: the first pool that is searched digit by digit
    (8, 16, 136, False),     # 128 for 127
])
def test_the_layer_that_exhausts_the_budget(rows, k, N, equal):
    """The best of a pool with more candidates than places, at the edges of the two ways it is done.  The
    scores are sums of two log-softmaxes, compared on the host in the same fp64 (gaps far above 1e-6)."""
    import torch
    import paper_2601_07353_amd as T
    V = 256
    rng = np.random.default_rng(7 * rows + k)
    x = rng.permuted(np.tile(np.arange(V, dtype=np.float32) * 0.0625, (N, 1)), axis=1) if not equal else np.full((N, V), -5, np.float32)
    if equal:
        x[0, :rows] = 5.0
        x[1:, :k] = 3.0
    else:
        x += rng.uniform(0.0, 0.03, size=(N, 1)).astype(np.float32) * (np.arange(V) % 7 == 3)
    logp = x.astype(np.float64) - np.logaddexp.reduce(x.astype(np.float64), axis=1, keepdims=True)
    best = lambda row, n: np.argsort(-x[row], kind="stable")[:n]
    first = best(0, max(k, rows))[:rows]
    pool = [(j, t, logp[0, first[j]] + logp[1 + j, t]) for j in range(rows) for t in best(1 + j, k)]
    scores = np.array([s for _, _, s in pool])
    places = N - 1 - rows
    if not equal:
        ordered = np.sort(scores)[::-1]
        assert ordered[places - 1] - ordered[places] > 1e-5, "the host cannot tell these apart"
    keep = sorted(np.argsort(-np.round(scores, 9), kind="stable")[:places])
    token = list(first) + [pool[i][1] for i in keep]
    parent = [0] * rows + [1 + pool[i][0] for i in keep]

    logits = torch.from_numpy(x).cuda().reshape(1, N, V)
    got = [build(logits, N, k, 2, ahead, K_init=rows, mu=1e-30) for ahead in (True, False)]
    st = T.TreeState(1, N)
    cand = T.Candidates(1, st.N_pad, k)
    ws = T.make_expand_workspace(1, st.N_pad, V, k, T.TALON_DTYPE_F32)
    T.talon_tree_init(st, torch.zeros(1, dtype=torch.int32).cuda())
    for d in range(2):
        T.talon_expand_layer(logits, st, k, cand, ws, layer=d)
        T.talon_select_budget(st, k, cand, 1e-30, rows, 1, 2)
    got.append({n: getattr(st, n).cpu().numpy() for n in ("token", "parent", "n_nodes")})
    for g in got:
        assert int(g["n_nodes"][0]) == N
        np.testing.assert_array_equal(g["token"][0, 1:N], token)
        np.testing.assert_array_equal(g["parent"][0, 1:N], parent)
