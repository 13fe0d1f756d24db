"""Alg. 2 with the candidate pool as the listing writes it (every token of every frontier row)
through talon_expand_literal, against the oracle.

The oracle runs with a per-row cap of N - 1: a layer never takes more than N - |T| <= N - 1
nodes, so that pool gives the uncapped tree (tests/test_oracle_pins.py checks that equivalence
against the full-vocabulary pool by brute force).  Seeds are admissible for that pool (every
cross-parent decision leaves a margin above the harness tolerance); topology, tokens, depths,
counters, status bits and the mask are then compared bit for bit, probabilities to 1e-5."""
import dataclasses

import numpy as np
import pytest

from tests import harness as H
from workloads import CONFIGS

pytestmark = pytest.mark.gpu

CASES = {
    # fp32 rows so flat that one parent receives more than 64 children: beyond the capped path
    "flat-f32-n200": dataclasses.replace(CONFIGS["c1"], name="literal-flat", V=4099, N=200, Dmax=8, K=4,
                                         recipe=("gauss", 0.3, 0.5)),
    # tiny fp32 shape, ragged vocabulary, K_init larger than the per-row cap of the fast path's config
    "tiny-f32": dataclasses.replace(CONFIGS["c1"], name="literal-tiny", V=1021, N=16, K=3),
    # Qwen3-8B-shaped rows, N = 128: one low-temperature and one high-temperature sequence
    "qwen-bf16-n128": dataclasses.replace(CONFIGS["c3"], name="literal-c3", B=2,
                                          recipe=(("gauss", 6.0, 8.0), ("gauss", 0.5, 1.0))),
    # the stress recipe (Zipf-peaked and near-uniform rows), N = 256, three sequences
    "zipf-bf16-n256": dataclasses.replace(CONFIGS["c5"], name="literal-n256", B=3, V=32003),
}


def _case(cfg, init_layers=1, layer_by_layer=False):
    cap = cfg.N - 1
    seeds, trees = [], []
    for b in range(cfg.B):
        s, _ = H.find_admissible_seed(cfg, b, cfg.seed + 100 * b, cap=cap, init_layers=init_layers)
        seeds.append(s)
    pool = H.build_pool(cfg, seeds)
    roots = H.root_tokens(cfg)
    from oracle import talon_oracle as O
    masks = []
    for b in range(cfg.B):
        t = H.oracle_tree(cfg, pool[b], roots[b], init_layers=init_layers, cap=cap)
        trees.append(t)
        masks.append(O.build_tree_mask(t.parent))
    for roomy in ((False, True) if cfg.N_pad == 64 else (False,)):
        gpu = H.run_gpu_literal(cfg, pool, cfg.K, init_layers=init_layers, layer_by_layer=layer_by_layer, roomy_state=roomy)
        H.compare_tree(cfg, gpu, trees, check_rows=False)
        H.compare_mask(cfg, gpu, masks)
    return trees


@pytest.mark.parametrize("name", list(CASES))
def test_uncapped_pool_matches_the_oracle(name):
    trees = _case(CASES[name])
    fan = max(int(np.bincount(np.asarray(t.parent[1:]), minlength=t.n).max()) for t in trees)
    print(name, "largest fan-out", fan, "nodes", [t.n for t in trees])
    if name == "flat-f32-n200":
        assert fan > 64   # the case the capped path cannot build


def test_one_layer_per_call_and_two_top_k_layers():
    _case(CASES["qwen-bf16-n128"], init_layers=2, layer_by_layer=True)
    _case(CASES["tiny-f32"], init_layers=0, layer_by_layer=True)


@pytest.mark.parametrize("layer_by_layer", [False, True])
def test_small_trees_whose_rows_get_more_than_32_children(layer_by_layer):
    """Trees of at most 64 nodes are first built with a per-row cap of 32 and, when a selection
    kept the 32nd candidate of a row, again from the saved state with the cap N - 1.  Three
    sequences in one call: peaked rows (largest fan-out 5), flat rows where one parent gets 31
    children (the last count the first build may keep) and flat rows where one gets 36 (the
    second build, which then redoes all three).  With one call per layer the wide layer is the
    second call, so the state the second build goes back to is not the root's."""
    cfg = dataclasses.replace(CONFIGS["c1"], name="literal-wide-n60", B=3, V=4099, N=60, Dmax=8, K=2, mu=0.1,
                              recipe=(("gauss", 6.0, 8.0), ("gauss", 0.3, 0.5), ("gauss", 2.0, 2.5)))
    trees = _case(cfg, layer_by_layer=layer_by_layer)
    fans = [int(np.bincount(np.asarray(t.parent[1:]), minlength=t.n).max()) for t in trees]
    print("largest fan-out per sequence", fans, "nodes", [t.n for t in trees])
    assert fans[0] < 31 and fans[1] == 31 and fans[2] > 32
    # the same recipes one sequence at a time (other rows: fan-outs 5, 45, 38): a call whose first build stands, two whose second runs
    for b in range(3):
        one = dataclasses.replace(cfg, name="literal-wide-n60-%d" % b, B=1, recipe=cfg.recipe[b], seed=cfg.seed + 100 * b)
        _case(one, layer_by_layer=layer_by_layer)


@pytest.mark.parametrize("dtype,V", [("f32", 40001), ("bf16", 70001)])
def test_rows_streamed_in_parts(dtype, V):
    """A layer of a few rows leaves compute units idle, and its rows are streamed in parts by
    several workgroups (four here: two rows per sequence, at least 2048 vectors per part).
    Second layer of the three sequences: rows of which every token passes the gate (every part
    cuts to the limit of 197, the merge selects among 4 x 197 survivors); rows of which 320-380
    pass (f32: no part overflows, the merge selects) or about 60 (bf16: the merge copies); rows
    that the scan's 16 best settle (nothing is streamed)."""
    cfg = dataclasses.replace(CONFIGS["c1"], name="literal-parts", B=3, V=V, logits_dtype=dtype, N=200, Dmax=6, K=2, mu=0.05,
                              recipe=(("gauss", 0.05, 0.1), ("gauss", 1.6, 1.9), ("gauss", 6.0, 8.0)))
    trees = _case(cfg)
    fans = [int(np.bincount(np.asarray(t.parent[1:]), minlength=t.n).max()) for t in trees]
    print("largest fan-out per sequence", fans, "nodes", [t.n for t in trees])
    assert fans[0] > 190 and fans[1] >= 64 and fans[2] < 16
    _case(cfg, layer_by_layer=True)


def test_capped_path_agrees_where_its_cap_suffices():
    """N = 60, k = 59: the fast path's tree is the uncapped tree, so both entry points must
    produce the same arrays, bit for bit (probabilities included: same arithmetic)."""
    cfg = dataclasses.replace(CONFIGS["c2"], name="c2-cap59", K=59, V=32003)
    seeds = [H.find_admissible_seed(cfg, 0, cfg.seed, K_init=10)[0]]
    pool = H.build_pool(cfg, seeds)
    fast = H.run_gpu_step(cfg, seeds=seeds, pool=pool, with_attention=False, K_init=10)
    lit = H.run_gpu_literal(cfg, pool, 10)
    n = int(fast["n_nodes"][0])
    assert int(lit["n_nodes"][0]) == n
    for name in ("token", "parent", "depth", "prob", "logp"):
        np.testing.assert_array_equal(lit[name][0, :n], fast[name][0, :n], err_msg=name)
    for name in ("status", "depth_cur", "frontier_begin", "frontier_count"):
        assert int(lit[name][0]) == int(fast[name][0]), name
    np.testing.assert_array_equal(lit["mask"][0], fast["mask"][0])


# ----------------------------------------------------------------------------- degenerate rows
def _compare_pool(cfg, make_pool, need_margin=True, **kw):
    """make_pool(attempt) -> pool.  With need_margin the first pool that leaves every cross-parent
    decision a margin is used (the test fails if none of 16 does); otherwise make_pool(0)."""
    from oracle import talon_oracle as O
    roots = H.root_tokens(cfg)
    if need_margin:
        pool, trees = H.admissible_pool(cfg, make_pool, cap=max(cfg.N - 1, 1), **kw)
    else:
        pool = make_pool(0)
        trees = [H.oracle_tree(cfg, pool[b], roots[b], cap=max(cfg.N - 1, 1), **kw) for b in range(cfg.B)]
    # trees of at most 64 nodes: once through the call's shortcut, once kept on the general path
    for roomy in ((False, True) if cfg.N_pad == 64 else (False,)):
        gpu = H.run_gpu_literal(cfg, pool, cfg.K, roomy_state=roomy, **kw)
        H.compare_tree(cfg, gpu, trees, check_rows=False)
        H.compare_mask(cfg, gpu, [O.build_tree_mask(t.parent) for t in trees])
    return gpu, trees


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_constant_rows_every_candidate_ties(dtype):
    """Every logit equal: all scores of a layer tie exactly, in any arithmetic.  The order
    (parent ascending, token ascending) must decide: the first child of the root receives the
    whole remaining budget, 114 children with tokens 0..113."""
    from tests.test_gpu_parity import custom_pool, small
    cfg = small(name="lit-const", V=20011, logits_dtype=dtype, K=5, N=120, Dmax=6)
    pool = custom_pool(cfg, lambda b, i: np.full(cfg.V, 1.5))
    gpu, _ = _compare_pool(cfg, lambda attempt: pool, need_margin=False)
    assert list(gpu["token"][0, 1:6]) == [0, 1, 2, 3, 4]
    assert list(gpu["parent"][0, 6:120]) == [1] * 114
    assert list(gpu["token"][0, 6:120]) == list(range(114))


def test_two_valued_rows_cut_inside_a_run_of_equal_logits():
    """Rows with two distinct values: the budget cut falls inside a long run of equal logits of
    one parent, after whole runs of its siblings."""
    from tests.test_gpu_parity import custom_pool, small
    cfg = small(name="lit-two", V=9001, logits_dtype="f32", K=3, N=150, Dmax=6, mu=0.5)

    def make_pool(attempt):
        def fill(b, i):
            x = np.full(cfg.V, 0.0)
            x[(7 * i) % 50::50] = 2.0 + (0.01 + 0.001 * attempt) * i   # 181 high entries, their level depends on the node
            return x
        return custom_pool(cfg, fill)

    _compare_pool(cfg, make_pool)


def test_sorted_rows_and_neg_inf_entries():
    from tests.test_gpu_parity import custom_pool, small
    cfg = small(name="lit-sorted", V=17003, logits_dtype="f32", K=8, N=90, Dmax=8)

    def make_pool(attempt):
        rng = np.random.default_rng(5 + attempt)

        def fill(b, i):
            if i % 3 == 0:
                return np.linspace(-3, 3, cfg.V) * (1 + 0.1 * i)
            if i % 3 == 1:
                return np.linspace(4, -4, cfg.V) * (1 + 0.05 * i)
            x = np.full(cfg.V, -np.inf)
            idx = rng.choice(cfg.V, size=5, replace=False)
            x[idx] = rng.normal(size=5)
            return x

        return custom_pool(cfg, fill)

    _compare_pool(cfg, make_pool)


def test_vocab_smaller_than_the_first_layer():
    from tests.test_gpu_parity import small
    cfg = small(name="lit-tinyv", V=8, logits_dtype="f32", K=12, N=40, Dmax=4, mu=1e-30)
    _compare_pool(cfg, lambda attempt: H.build_pool(cfg, [cfg.seed + attempt]))


def test_nan_row_sets_status_and_stops_sequence():
    from tests.test_gpu_parity import small
    cfg = small(name="lit-nan", V=5000, logits_dtype="f32", K=3, N=20, Dmax=6, B=2)
    seeds = [H.find_admissible_seed(cfg, 0, cfg.seed, cap=cfg.N - 1)[0], cfg.seed]
    pool = H.build_pool(cfg, seeds)
    pool[1, 2, 1234] = np.nan
    t = H.oracle_tree(cfg, pool[0], H.root_tokens(cfg)[0], cap=cfg.N - 1)
    assert t.margin > H.MARGIN_TOL
    for roomy in (False, True):      # the shortcut for small trees, then the general path
        gpu = H.run_gpu_literal(cfg, pool, cfg.K, roomy_state=roomy)
        assert int(gpu["status"][1]) & 4
        assert int(gpu["n_nodes"][1]) == 1 + cfg.K          # stopped after the layer that read the bad row
        assert int(gpu["frontier_count"][1]) == 0
        H.compare_tree(cfg, {k: v[:1] for k, v in gpu.items()}, [t], check_rows=False)


def test_budget_of_one_and_two():
    from tests.test_gpu_parity import small
    for N in (1, 2):
        cfg = small(name="lit-n%d" % N, V=2048, logits_dtype="bf16", K=4, N=N, Dmax=4)
        _compare_pool(cfg, lambda attempt: H.build_pool(cfg, [cfg.seed]), need_margin=False)


# ----------------------------------------------------------------------------- full sizes
def _full_size(cfg_name, oracle_seqs):
    """All sequences of a benchmark configuration through the uncapped call; the oracle builds the
    stated sequences in full, every sequence is checked for the properties any tree must have."""
    from oracle import talon_oracle as O
    from tests.test_gpu_full_size import structural_checks
    cfg = CONFIGS[cfg_name]
    cap = cfg.N - 1
    seeds = [cfg.seed] * cfg.B
    trees = {}
    for b in oracle_seqs:
        seeds[b], trees[b] = H.find_admissible_seed(cfg, b, cfg.seed, cap=cap)
    print("case", cfg.name, "uncapped, seeds", seeds, "oracle sequences", oracle_seqs, flush=True)
    pool = H.build_pool(cfg, seeds)
    gpu = H.run_gpu_literal(cfg, pool, cfg.K)
    for b in range(cfg.B):
        structural_checks(cfg, gpu, b)
    for b in oracle_seqs:
        t = trees[b]
        assert t.margin > H.MARGIN_TOL
        H.compare_tree(cfg, {k: v[b:b + 1] for k, v in gpu.items()}, [t], check_rows=False)
        np.testing.assert_array_equal(gpu["mask"][b], O.mask_to_words(O.build_tree_mask(t.parent), cfg.N_pad))


def test_c3_qwen3_8b_x4_full_size_uncapped():
    _full_size("c3", [0, 1, 2, 3])


def test_c5_stress_full_size_uncapped():
    _full_size("c5", list(range(16)))


def test_repeated_calls_on_one_workspace_agree():
    """Survivors are collected in whatever order the lanes claim their slots; the tree must not
    depend on it, nor on what an earlier call left in the workspace (a different, larger shape
    first, then the same call twenty times)."""
    import torch
    import paper_2601_07353_amd as T
    big = CASES["zipf-bf16-n256"]
    cfg = CASES["qwen-bf16-n128"]
    dt = T.TALON_DTYPE_BF16
    ws = T.make_literal_workspace(big.B, big.N_pad, big.V, dt)
    assert ws.numel() >= T.load_library().talon_literal_workspace_bytes(cfg.B, cfg.N_pad, cfg.V, dt)

    def run(c, pool_dev):
        st = T.TreeState(c.B, c.N)
        T.talon_tree_init(st, torch.from_numpy(H.root_tokens(c)).cuda())
        T.talon_expand_literal(pool_dev, st, c.Dmax, c.mu, c.K, 1, c.Dmax, ws)
        torch.cuda.synchronize()
        n = st.n_nodes.cpu().numpy()
        return [n] + [getattr(st, f).cpu().numpy() for f in ("token", "parent", "depth", "prob", "logp", "status")]

    run(big, H.to_device_logits(H.build_pool(big, [big.seed] * big.B)))
    dev = H.to_device_logits(H.build_pool(cfg, [cfg.seed, cfg.seed + 100]))
    first = run(cfg, dev)
    assert all(int(v) == cfg.N for v in first[0])
    for _ in range(20):
        again = run(cfg, dev)
        for x, y in zip(first, again):
            n = first[0]
            if x.ndim == 2:
                for b in range(cfg.B):
                    np.testing.assert_array_equal(x[b, :n[b]], y[b, :n[b]])
            else:
                np.testing.assert_array_equal(x, y)


def test_random_small_configurations():
    """Thirty seeded random shapes (vocabulary 8 to 60001, both logit types, N 2-256, K_init 1-19
    -- above 16 the top-K layers take the streaming route too --, 1-3 sequences, 0-2 top-K layers,
    four thresholds and recipes, depth cap from 1), alternately in one call and one call per
    layer.  Configurations whose oracle tree leaves no margin are skipped; most must run."""
    from oracle import talon_oracle as O
    from workloads import WorkloadConfig
    rng = np.random.default_rng(20260107)
    ran = 0
    for it in range(30):
        dtype = str(rng.choice(["f32", "bf16"]))
        V = int(rng.choice([8, 63, 500, 4099, 20000, 60001]))
        N = int(rng.integers(2, 257))
        K = int(rng.integers(1, 20))
        B = int(rng.integers(1, 4))
        init_layers = int(rng.integers(0, 3))
        mu = float(rng.choice([0.3, 0.03, 0.003, 1e-6]))
        rec = [("gauss", 0.5, 4.0), ("gauss", 0.05, 0.3), ("gauss", 4.0, 8.0), ("zipf_mix", 1.2, 0.05)][int(rng.integers(0, 4))]
        Dmax = int(rng.integers(1, 10))
        if B * ((N + 63) // 64 * 64) * V > 60e6:
            V = 4099
        cfg = WorkloadConfig("literal-random-%d" % it, B=B, V=V, logits_dtype=dtype, K=K, N=N, Dmax=Dmax, mu=mu,
                             Hq=4, Hkv=4, Dh=64, L=16, recipe=rec, seed=1000 + it)
        pool = H.build_pool(cfg, [cfg.seed + 7 * b for b in range(B)])
        roots = H.root_tokens(cfg)
        trees = [H.oracle_tree(cfg, pool[b], roots[b], init_layers=init_layers, cap=max(N - 1, 1)) for b in range(B)]
        if min(t.margin for t in trees) <= H.MARGIN_TOL:
            continue
        print("case", it, dtype, "V", V, "N", N, "K", K, "B", B, "init", init_layers, "mu", mu, rec, "Dmax", Dmax, flush=True)
        for roomy in ((False, True) if cfg.N_pad == 64 else (False,)):
            gpu = H.run_gpu_literal(cfg, pool, K, init_layers=init_layers, layer_by_layer=bool(it % 2), roomy_state=roomy)
            H.compare_tree(cfg, gpu, trees, check_rows=False)
            H.compare_mask(cfg, gpu, [O.build_tree_mask(t.parent) for t in trees])
        ran += 1
    assert ran >= 24


def test_dense_frontier_batches_with_padded_rows():
    """The layout a serving loop has: after every layer the draft model's logits exist for the
    new frontier only, as a dense batch [B][frontier rows][padded row] (TALON_ROWS_BY_FRONTIER,
    row stride larger than the vocabulary, values in the padding that would win any maximum).
    One uncapped call per layer on a freshly gathered batch must build the oracle's tree."""
    import torch
    import paper_2601_07353_amd as T
    from tests.test_gpu_parity import small
    cfg = small(name="literal-dense", V=20011, logits_dtype="bf16", K=6, N=150, Dmax=9, B=3,
                recipe=(("gauss", 4.0, 8.0), ("gauss", 0.5, 1.0), ("gauss", 2.0, 6.0)))
    cap = cfg.N - 1
    seeds = [H.find_admissible_seed(cfg, b, cfg.seed + 100 * b, cap=cap)[0] for b in range(cfg.B)]
    pool = H.build_pool(cfg, seeds)
    roots = H.root_tokens(cfg)
    trees = [H.oracle_tree(cfg, pool[b], roots[b], cap=cap) for b in range(cfg.B)]
    pool_dev = H.to_device_logits(pool)                      # [B][N_pad][V], only used to gather from
    stride = (cfg.V + 8 + 63) // 64 * 64
    st = T.TreeState(cfg.B, cfg.N)
    ws = T.make_literal_workspace(cfg.B, st.N_pad, cfg.V, T.TALON_DTYPE_BF16)
    T.talon_tree_init(st, torch.from_numpy(roots).cuda())
    for _ in range(cfg.Dmax):
        begin = st.frontier_begin.cpu().numpy()
        count = st.frontier_count.cpu().numpy()
        done = (st.status.cpu().numpy() & 3) != 0
        if done.all():
            break
        fmax = max(1, int(count.max()))
        dense = torch.full((cfg.B, fmax, stride), 30000.0, dtype=torch.bfloat16, device="cuda")
        for b in range(cfg.B):
            if not done[b]:
                dense[b, :count[b], :cfg.V] = pool_dev[b, begin[b]:begin[b] + count[b]]
        T.talon_expand_literal(dense, st, 1, cfg.mu, cfg.K, 1, cfg.Dmax, ws, row_mode=T.TALON_ROWS_BY_FRONTIER,
                               vocab=cfg.V)
        torch.cuda.synchronize()
    n = st.n_nodes.cpu().numpy()
    for b, t in enumerate(trees):
        assert int(n[b]) == t.n
        np.testing.assert_array_equal(st.token[b, :t.n].cpu().numpy(), np.asarray(t.token, dtype=np.int32))
        np.testing.assert_array_equal(st.parent[b, :t.n].cpu().numpy(), np.asarray(t.parent, dtype=np.int32))
        np.testing.assert_allclose(np.exp(st.logp[b, :t.n].cpu().numpy()), t.confidence(), rtol=H.PROB_RTOL, atol=0)
    assert max(int(np.bincount(np.asarray(t.parent[1:])).max()) for t in trees) > cfg.K


# B, V, dtype, N, K_init, init_layers, mu, rows: one row kind per sequence in turn
AHEAD_SHAPES = [
    (1, 8, "f32", 12, 3, 1, 0.03, "mixed"),            # fewer tokens than the 16 that a scan ranks
    (1, 17, "bf16", 64, 20, 1, 1e-6, "flat"),          # top-K layer wider than that; every token passes the gate
    (2, 4099, "f32", 33, 16, 0, 0.03, "mixed"),        # no top-K layer: the root's row is read again
    (3, 20011, "bf16", 60, 10, 1, 0.03, "mixed"),
    (2, 5003, "f32", 130, 4, 2, 0.1, "equal"),         # every score ties; one part of a row holds all its children
    (70, 1021, "bf16", 20, 5, 1, 0.03, "mixed"),       # more sequences than a helper polls at once and than helpers
    (4, 151936, "bf16", 128, 8, 1, 0.03, "mixed"),     # eight parts per row
    (2, 40001, "f32", 256, 2, 1, 0.003, "flat"),       # two rows share 253 children
    (16, 60001, "bf16", 250, 16, 1, 0.03, "mixed"),    # several rounds of rows, helpers from the start
    (16, 100003, "bf16", 250, 16, 1, 0.03, "mixed"),   # ... many of them
    (2, 20011, "bf16", 48, 47, 1, 0.03, "mixed"),      # the first layer spends the budget: its row is read again
    (2, 30011, "f32", 128, 127, 1, 0.03, "mixed"),
    (8, 30011, "bf16", 220, 8, 1, 0.03, "flat"),       # the budget is sure to be spent before the rows are read again: late helpers
    (5, 20002, "f32", 200, 8, 1, 0.03, "steps"),       # ... and it is not, though all 16 best pass: 20 tokens of a row do
]


@pytest.mark.parametrize("shape", AHEAD_SHAPES, ids=lambda s: "-".join(str(x) for x in s))
@pytest.mark.parametrize("steps", [(24,), (4, 24)])
def test_rows_scanned_ahead_give_the_layered_trees(shape, steps):
    """talon_expand_literal_ahead against talon_expand_literal, in one call and continued in the
    middle of the trees, with a sequence that is finished from the start and one that has a bad row."""
    import ctypes
    import torch
    import paper_2601_07353_amd as T
    B, V, dtype, N, K_init, init_layers, mu, kind = shape
    print("case", shape, steps, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(V * 1000 + N)
    dt, code = (torch.float32, T.TALON_DTYPE_F32) if dtype == "f32" else (torch.bfloat16, T.TALON_DTYPE_BF16)
    stride = (V + 7) // 8 * 8
    st = [T.TreeState(B, N) for _ in range(2)]
    P = st[0].N_pad
    pool = torch.full((B, P, stride), 60.0, dtype=dt, device="cuda")
    for b in range(B):
        scale = torch.rand(P, 1, generator=g, device="cuda")
        scale = 0.3 + 0.2 * scale if kind == "flat" or (kind == "mixed" and b % 3 == 1) else 0.5 + 7.5 * scale
        pool[b, :, :V] = (torch.randn(P, V, generator=g, device="cuda") * scale).to(dt) if kind != "equal" else 1.5
        if kind == "steps":
            pool[b, :, :V] = (pool[b, :, :V] * 0.01 - 3.0).to(dt)
            pool[b, :, 100 * b:100 * b + 40:2] = (3.0 + 0.001 * torch.arange(20, device="cuda")).to(dt)
    if B > 2:
        pool[2, 1, V // 2] = float("nan")
    logits = pool[:, :, :V]
    roots = torch.arange(B, dtype=torch.int32, device="cuda")
    ws = T.make_literal_workspace(B, P, V, code)
    lib = T.load_library()
    lib.talon_expand_literal.restype = lib.talon_expand_literal_ahead.restype = ctypes.c_int
    for i, s in enumerate(st):
        T.talon_tree_init(s, roots)
        if B > 1:
            s.status[1] = T.TALON_STATUS_DONE_DEPTH
        ws.fill_(0xA5)
        for layers in steps:
            if i == 0:
                rc = lib.talon_expand_literal(logits.data_ptr(), code, stride, stride * P, T.TALON_ROWS_BY_NODE, layers, ctypes.byref(s.c),
                                              V, mu, K_init, init_layers, 24, ws.data_ptr(), ws.numel(), None)
            else:
                rc = lib.talon_expand_literal_ahead(logits.data_ptr(), code, stride, stride * P, N - 1, layers, ctypes.byref(s.c),
                                                    V, mu, K_init, init_layers, 24, ws.data_ptr(), ws.numel(), None)
            assert rc == T.TALON_OK
            torch.cuda.synchronize()
    # the ahead form leaves its counters at zero, as the other forms of one workspace want them
    assert not ws[:(B * P * 4 + 255) // 256 * 256].any()
    want, got = ({k: getattr(s, k).cpu().numpy() for k in ("n_nodes", "status", "depth_cur", "frontier_begin", "frontier_count",
                                                          "token", "parent", "depth", "prob", "logp")} for s in st)
    for name in ("n_nodes", "status", "depth_cur", "frontier_begin", "frontier_count", "token", "parent", "depth"):
        np.testing.assert_array_equal(got[name], want[name], err_msg=name)
    if B > 2:
        assert int(want["status"][2]) & T.TALON_STATUS_BAD_ROW and int(want["n_nodes"][1]) == 1
    # sums of the same fp32 exponentials, grouped otherwise (at most 32 in single precision either way): a few
    # of their roundings, 2^-24 each
    np.testing.assert_allclose(got["logp"], want["logp"], rtol=0, atol=24 * 4 * 2.0 ** -24)
    # ... and for a small probability the log-probability is rounded to single precision (2^-24 of it), and so is its product
    # with log2(e), before the exponential: a last bit that differs moves either, on both sides
    small = 4 * np.abs(np.log(np.maximum(want["prob"], 1e-37), dtype=np.float64)) * 2.0 ** -24
    assert (np.abs(got["prob"].astype(np.float64) - want["prob"]) <= (16 * 2.0 ** -24 + small) * want["prob"]).all()


@pytest.mark.parametrize("N", [60, 130])
def test_any_number_of_layers_means_the_whole_loop(N):
    """Trees continued below the root with the largest number a caller can pass: layered, ahead and through the
    Python call the oracle's trees."""
    import ctypes
    import torch
    import paper_2601_07353_amd as T
    from tests.test_gpu_parity import small
    cfg = small(name="literal-all-layers", V=4099, logits_dtype="bf16", K=3, N=N, Dmax=9, B=2, recipe=("gauss", 7.0, 9.0))
    pool, trees = H.admissible_pool(cfg, lambda i: H.build_pool(cfg, [cfg.seed + 10 * i + b for b in range(cfg.B)]), cap=N - 1)
    assert min(len(t.layers) for t in trees) > 3
    dev = H.to_device_logits(pool)
    lib = T.load_library()
    lib.talon_expand_literal_ahead.restype = ctypes.c_int
    for how in ("layered", "ahead", "python"):
        st = T.TreeState(cfg.B, cfg.N)
        ws = T.make_literal_workspace(cfg.B, st.N_pad, cfg.V, T.TALON_DTYPE_BF16)
        T.talon_tree_init(st, torch.from_numpy(H.root_tokens(cfg)).cuda())
        for layers in (1, 2 ** 31 - 1):
            args = (layers, ctypes.byref(st.c), cfg.V, cfg.mu, cfg.K, 1, cfg.Dmax, ws.data_ptr(), ws.numel(), None)
            at = (dev.data_ptr(), T.TALON_DTYPE_BF16, dev.stride(1), dev.stride(0))
            if how == "layered":
                assert lib.talon_expand_literal(*at, T.TALON_ROWS_BY_NODE, *args) == T.TALON_OK
            elif how == "ahead":
                assert lib.talon_expand_literal_ahead(*at, N - 1, *args) == T.TALON_OK
            else:
                T.talon_expand_literal(dev, st, layers, cfg.mu, cfg.K, 1, cfg.Dmax, ws)
        for b, t in enumerate(trees):
            assert int(st.n_nodes[b]) == t.n, (how, b)
            np.testing.assert_array_equal(st.token[b, :t.n].cpu().numpy(), np.asarray(t.token, dtype=np.int32))
            np.testing.assert_array_equal(st.parent[b, :t.n].cpu().numpy(), np.asarray(t.parent, dtype=np.int32))


@pytest.mark.parametrize("dtype,V", [("bf16", 40003), ("bf16", 20007), ("bf16", 70), ("f32", 20001), ("f32", 4099), ("f32", 18)])
def test_rows_that_end_with_the_buffer(dtype, V):
    """The last row of the last sequence ends at its last token, and the tokens behind the row's last whole
    16-byte vector are among those that a second reading finds: the trees of a padded buffer, layered and ahead."""
    import ctypes
    import torch
    import paper_2601_07353_amd as T
    print("case", dtype, V, flush=True)
    B, N, K_init = 2, 100, 40
    dt, code = (torch.float32, T.TALON_DTYPE_F32) if dtype == "f32" else (torch.bfloat16, T.TALON_DTYPE_BF16)
    stride, P = (V + 7) // 8 * 8, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(V)
    padded = torch.full((B, P, stride), 60.0, dtype=dt, device="cuda")
    padded[:, :, :V] = (torch.randn(B, P, V, generator=g, device="cuda") * 0.1).to(dt)
    padded[:, ::2, V - 2:V] = 0.9      # high enough to be chosen, too low for a row's 16 best
    padded[:, ::2, :20] = 1.0
    whole = torch.empty((B * P - 1) * stride + V, dtype=dt, device="cuda")
    exact = torch.as_strided(whole, (B, P, V), (P * stride, stride, 1))
    exact.copy_(padded[:, :, :V])
    lib = T.load_library()
    lib.talon_expand_literal.restype = lib.talon_expand_literal_ahead.restype = ctypes.c_int
    ws = T.make_literal_workspace(B, P, V, code)
    got = []
    for logits in (padded, exact):
        for ahead in (False, True):
            st = T.TreeState(B, N)
            T.talon_tree_init(st, torch.arange(B, dtype=torch.int32, device="cuda"))
            fn, row_arg = (lib.talon_expand_literal_ahead, P) if ahead else (lib.talon_expand_literal, T.TALON_ROWS_BY_NODE)
            assert fn(logits.data_ptr(), code, stride, stride * P, row_arg, 24, ctypes.byref(st.c), V, 0.03, K_init, 1, 24, ws.data_ptr(),
                      ws.numel(), None) == T.TALON_OK
            got.append({k: getattr(st, k).cpu().numpy() for k in ("n_nodes", "token", "parent", "depth", "status")})
    for other in got[1:]:
        for k, v in got[0].items():
            np.testing.assert_array_equal(other[k], v, err_msg=k)
    assert (got[0]["token"][0, 1:N] >= V - 2).sum() >= 2 and (got[0]["n_nodes"] == N).all()


@pytest.mark.parametrize("microseconds", [0, 1, 2, 3, 5])
def test_a_wait_that_runs_out_leaves_trees_to_go_on_from(microseconds):
    """The bound of the waits reaches the launch that scans ahead: a call whose bound runs out (here a short one, from
    the host) ends with every sequence ABORTED after a whole layer; with the bit cleared another call finishes the trees."""
    import ctypes
    import torch
    import paper_2601_07353_amd as T
    B, V, N, stride = 4, 70001, 200, 70008
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    scale = torch.tensor([6.0, 0.4, 4.0, 0.5], device="cuda")[:, None, None]     # two sequences whose rows are read again
    logits = (torch.randn(B, 256, stride, generator=g, device="cuda") * scale).bfloat16()[:, :, :V]
    ws = T.make_literal_workspace(B, 256, V, T.TALON_DTYPE_BF16)
    st = [T.TreeState(B, N) for _ in range(2)]
    for s in st:
        T.talon_tree_init(s, torch.arange(B, dtype=torch.int32, device="cuda"))
    for _ in range(16):                                                          # (layer by layer: nothing waits)
        T.talon_expand_literal(logits, st[0], 1, 0.03, 8, 1, 16, ws)
    T.talon_set_spin_limit_us(microseconds)
    try:
        T.talon_expand_literal(logits, st[1], 16, 0.03, 8, 1, 16, ws)
        torch.cuda.synchronize()
    finally:
        T.talon_set_spin_limit_us(200000)
    want = {k: getattr(st[0], k).cpu().numpy() for k in ("n_nodes", "status", "token", "parent", "depth", "depth_cur")}
    cut = {k: getattr(st[1], k).cpu().numpy().copy() for k in want}
    aborted = (cut["status"] & T.TALON_STATUS_ABORTED) != 0
    print("bound", microseconds, "aborted", aborted, "nodes", cut["n_nodes"], "of", want["n_nodes"], flush=True)
    assert aborted.all() or not aborted.any()
    if microseconds == 0:
        assert aborted.all()
    for b in range(B):
        n = int(cut["n_nodes"][b])
        for k in ("token", "parent", "depth"):
            np.testing.assert_array_equal(cut[k][b, :n], want[k][b, :n], err_msg=k)
        assert n == int(want["n_nodes"][b]) or int(want["depth"][b, n]) == int(cut["depth_cur"][b]) + 1     # whole layers
    st[1].status &= ~T.TALON_STATUS_ABORTED
    T.talon_expand_literal(logits, st[1], 16, 0.03, 8, 1, 16, ws)
    for k, v in want.items():
        got = getattr(st[1], k).cpu().numpy()
        np.testing.assert_array_equal(got if got.ndim == 1 else got[:, :N], v if v.ndim == 1 else v[:, :N], err_msg=k)
