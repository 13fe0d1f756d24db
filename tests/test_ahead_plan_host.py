"""Launch plan of the scan ahead of the tree, evaluated on the host (no GPU)."""
import random

from tests import plan_host as P


def shapes(count, seed):
    r = random.Random(seed)
    for _ in range(count):
        k = r.choice([1, 2, 4, 8, 10, 16, 31, 64])
        yield dict(B=r.randint(1, 256), N=r.randint(2, min(256, 4096 // k + 1)), vocab=int(2 ** r.uniform(0, 18)),
                   dtype=r.choice(["f32", "bf16"]), k=k, K_init=r.choice([1, k, r.randint(1, 64)]), init_layers=r.randint(0, 3),
                   max_depth=r.choice([1, 2, 3, 4, 6, 12, 24, 256]))


def test_every_row_a_tree_can_expand_is_scanned():
    """Selectors wait for the rows of their frontier, so the scan has to cover every row that any tree of
    these parameters expands: trees that keep as many candidates per layer as they may, or fewer at random."""
    r = random.Random(1)
    for c in shapes(4000, 2):
        rows = P.ahead_plan(**c)["rows"]
        assert 1 <= rows <= c["N"] - 1
        for greedy in (True, False, False, False):
            n, frontier, expanded = 1, 1, 0
            for d in range(c["max_depth"]):
                expanded += frontier
                most = min(frontier * c["k"], c["N"] - n)
                if d < c["init_layers"]:
                    most = min(most, c["K_init"])
                frontier = most if greedy else r.randint(1, most)
                n += frontier
                if n >= c["N"]:
                    break
            assert expanded <= rows, (c, rows, expanded)


def test_runs_cover_rows_in_whole_blocks():
    for c in shapes(4000, 3):
        p = P.ahead_plan(**c)
        assert 0 <= p["head"] <= p["rows"], (c, p)
        for chunks in (p["chunks_head"], p["chunks"]):
            per_run = -(-p["blocks"] // chunks)
            assert 1 <= chunks <= p["blocks"] and (chunks - 1) * per_run < p["blocks"], (c, p)
        items = c["B"] * (p["head"] * p["chunks_head"] + (p["rows"] - p["head"]) * p["chunks"])
        assert 1 <= p["scanners"] <= min(items, 1024), (c, p)


def test_a_depth_cap_bounds_the_rows_that_are_scanned():
    # 1 + 8 rows of 199, 1 + 16 + 64; a cap that no layer reaches changes nothing
    assert P.ahead_plan(4, 200, 128256, "bf16", 8, 2)["rows"] == 9
    assert P.ahead_plan(4, 200, 128256, "bf16", 8, 3)["rows"] == 73
    assert P.ahead_plan(4, 200, 128256, "bf16", 8, 3, K_init=2)["rows"] == 1 + 2 + 16
    assert P.ahead_plan(4, 200, 128256, "bf16", 8, 24)["rows"] == 199
    # ... and the rows that are left are cut as finely as the grid allows
    assert P.ahead_plan(4, 200, 128256, "bf16", 8, 2)["chunks"] == 16


def test_trees_with_nothing_to_scan_ahead_are_built_layer_by_layer():
    layered = lambda *a, **kw: bool(P.ahead_plan(*a, **kw)["layered"])
    assert layered(9, 148, 151936, "bf16", 2, 1)                      # one layer
    assert not layered(9, 148, 151936, "bf16", 2, 1, init_layers=0)   # ... selected by the gate
    assert layered(32, 17, 151936, "bf16", 16, 12)                    # the first layer spends the budget
    assert not layered(32, 18, 32000, "f32", 16, 12)
    assert not layered(4, 17, 151936, "f32", 16, 12)                  # ... but its rows have 38 blocks, in 13 runs
    assert layered(1, 17, 151936, "f32", 16, 12)                      # ... in 38
    assert not layered(1, 17, 32000, "bf16", 16, 12, init_layers=0)   # ... may or may not, without a top-K layer
    assert layered(16, 200, 151936, "bf16", 16, 3)                    # three layers, 60 blocks per scanner
    assert not layered(8, 128, 151936, "bf16", 8, 3)                  # ... 11
    assert not layered(16, 200, 151936, "bf16", 16, 4)
    for B, N, V, k, D in [(1, 16, 1024, 2, 6), (1, 60, 128256, 10, 12), (4, 128, 151936, 8, 16), (16, 256, 151936, 16, 24)]:
        assert not layered(B, N, V, "bf16", k, D)


# B, N, vocabulary, layers, K_init, layer by layer?: measured on both sides of each line
UNCAPPED = [
    (1, 60, 128256, 3, 8, True), (1, 60, 128256, 4, 8, False),                     # layers
    (16, 250, 64000, 4, 8, True), (16, 250, 64000, 5, 8, False),                   # ... against blocks per scanner
    (8, 250, 151936, 5, 8, True), (8, 250, 151936, 6, 8, False),
    (16, 250, 151936, 8, 8, True), (16, 250, 151936, 12, 8, False),
    (8, 33, 128256, 6, 32, True), (8, 36, 128256, 6, 35, False),                   # the first layer spends the budget
    (1, 128, 128256, 6, 127, False), (1, 250, 20000, 6, 249, True), (16, 100, 128256, 6, 99, True), (4, 100, 128256, 6, 99, False),
]


def test_uncapped_calls_go_the_way_that_was_faster():
    for B, N, vocab, layers, K_init, layered in UNCAPPED:
        assert P.literal_layered(B, N, vocab, "bf16", layers, K_init) == layered, (B, N, vocab, layers, K_init)
    # without a top-K layer, rows decide whether the first layer spends the budget
    assert not P.literal_layered(8, 33, 128256, "bf16", 6, 32, init_layers=0)
    # no product overflows
    assert P.literal_layered(256, 256, 2 ** 31 - 1, "f32", 255) and not P.literal_layered(1, 256, 1000, "f32", 2 ** 31 - 1)
