"""Launch plan of tree attention, evaluated on the host (no GPU)."""
import random

import pytest

from tests import plan_host as P


def shapes(count, seed):
    r = random.Random(seed)
    for _ in range(count):
        Hkv = r.choice([1, 2, 3, 4, 8, 16])
        yield (r.randint(1, 70), 64 * r.randint(1, 4), Hkv * r.choice([1, 2, 3, 4, 8, 16]), Hkv, r.choice([64, 128]),
               int(2 ** r.uniform(0, 17.5)) - 1)


def tiles_of(N_pad, L):
    return (L + 63) // 64 + N_pad // 64


def filling(B, N_pad, Hq, Hkv, L):
    """Wavefronts and splits that fill the chip: 256 workgroups of 8 wavefronts or 512 of 4, rounded up, with at
    least four key tiles a split."""
    rows = N_pad * (Hq // Hkv)
    waves = 8 if rows >= 512 else 4
    pairs = B * Hkv * (-(-rows // (32 * waves)))
    tiles = tiles_of(N_pad, L)
    want = max(1, min(-(-(256 if waves == 8 else 512) // pairs), max(1, tiles // 4)))
    run = -(-tiles // want)
    return waves, -(-tiles // run)


@pytest.mark.parametrize("part", [1.0, 0.5, 0.0])
def test_a_plan_covers_every_key_and_fits_its_workspace(part):
    for B, N_pad, Hq, Hkv, Dh, L in shapes(3000, 1):
        least = P.least_workspace(B, N_pad, Hq, Hkv, Dh, L)
        nbytes = least + int(part * max(0, P.attention_plan(B, N_pad, Hq, Hkv, Dh, L)["bytes"] - least))
        p = P.attention_plan(B, N_pad, Hq, Hkv, Dh, L, nbytes)
        where = (B, N_pad, Hq, Hkv, Dh, L, nbytes, p)
        tiles, rows = tiles_of(N_pad, L), N_pad * (Hq // Hkv)
        assert p["waves"] in (4, 8) and p["row_tiles"] == -(-rows // (32 * p["waves"])), where
        assert p["split_likely"] == -(-tiles // p["run_bound"]) <= p["split_max"], where
        assert p["capacity_per_head"] >= B * p["row_tiles"] * p["split_likely"], where
        assert p["bytes"] <= max(nbytes, 256), where
        assert p["balance"] == (p["split_max"] > p["split_likely"]), where
        staged = p["split_max"] > 1
        assert p["partial"] == (B * Hkv * p["row_tiles"] * p["split_max"] * 32 * p["waves"] * (2 * Dh + 8) if staged else 256), where


def test_rows_the_filling_plan_leaves_in_registers_are_not_staged():
    """Staged partial results are rounded to bf16.  Where one run per row tile fills the chip, a row goes from
    fp32 registers to the output, and no other plan (more splits, unequal prefixes sharing the grid) may stage it."""
    seen = 0
    for B, N_pad, Hq, Hkv, Dh, L in shapes(4000, 2):
        if filling(B, N_pad, Hq, Hkv, L)[1] > 1:
            continue
        p = P.attention_plan(B, N_pad, Hq, Hkv, Dh, L)
        assert p["split_max"] == 1 and not p["balance"], (B, N_pad, Hq, Hkv, Dh, L, p)
        seen += 1
    assert seen > 500


def test_one_filling_run_stays_one_run():
    """The kernels keep a sequence of at most run_single key tiles in one run (one rounding to bf16): the run
    length of the plan that fills the chip, none where that plan has a single run for everybody."""
    for B, N_pad, Hq, Hkv, Dh, L in shapes(3000, 3):
        splits = filling(B, N_pad, Hq, Hkv, L)[1]
        want = -(-tiles_of(N_pad, L) // splits) if splits > 1 else 0
        assert P.attention_plan(B, N_pad, Hq, Hkv, Dh, L)["run_single"] == want, (B, N_pad, Hq, Hkv, Dh, L)
    assert (P.attention_plan(3, 192, 64, 16, 64, 793)["run_single"], P.attention_plan(5, 256, 32, 4, 64, 2000)["run_single"]) == (8, 18)


def test_plans_that_leave_the_filling_one_share_the_grid_among_unequal_prefixes():
    """A plan that is cheaper for full-length prefixes only loses to the filling one when prefixes are unequal
    (3 sequences of 4525, 6643 and 9213 of 14916 keys: runs of 48 tiles on 256 workgroups took 118 us, runs of 79
    on 128 took 95), so it has to bring the balancing, and the query the workspace for it."""
    seen = 0
    for B, N_pad, Hq, Hkv, Dh, L in shapes(4000, 4):
        waves, splits = filling(B, N_pad, Hq, Hkv, L)
        p = P.attention_plan(B, N_pad, Hq, Hkv, Dh, L)
        if B == 1 or p["split_likely"] == 1 or (p["waves"], p["split_likely"]) == (waves, splits) or p["run_bound"] < 8:
            continue
        seen += 1
        assert p["balance"] and p["split_max"] == 2 * p["split_likely"], (B, N_pad, Hq, Hkv, Dh, L, p)
    assert seen > 200


def test_long_prefixes_of_few_heads_fill_the_chip():
    """The number of splits has no cap of its own: 64 runs of a 262144-key prefix leave three quarters of the chip
    idle (one KV head of 64 query rows: 93 us, 57 with 228 runs).  The filling plan is always a candidate."""
    for Hkv, G, L in [(1, 1, 131072), (1, 4, 131072), (2, 2, 131072), (1, 1, 262144), (2, 4, 262144)]:
        for Dh in (64, 128):
            assert P.attention_plan(1, 64, Hkv * G, Hkv, Dh, L)["split_likely"] > 64, (Hkv, G, Dh, L)
    for B, N_pad, Hq, Hkv, Dh, L in shapes(3000, 5):
        waves, splits = filling(B, N_pad, Hq, Hkv, L)
        p = P.attention_plan(B, N_pad, Hq, Hkv, Dh, L)
        us = P.plan_us(B, N_pad, Hq, Hkv, Dh, L, p["waves"], p["split_likely"])
        assert us <= P.plan_us(B, N_pad, Hq, Hkv, Dh, L, waves, splits) + 1e-9, (B, N_pad, Hq, Hkv, Dh, L, p)


def device_run(p, n_list, G, L_list):
    """The run length the balanced kernels work out from the lengths of a batch."""
    tiles = [-(-L // 64) + -(-n // 64) for n, L in zip(n_list, L_list)]
    row_tiles = [-(-n * G // (32 * p["waves"])) for n in n_list]
    for run in range(max(4, -(-max(tiles) // p["split_max"])), p["run_bound"]):
        if sum(r * (1 if t <= p["run_single"] else -(-t // run)) for r, t in zip(row_tiles, tiles)) <= p["capacity_per_head"]:
            return run
    return p["run_bound"]


def test_the_balanced_batches_of_the_gpu_tests_reach_all_four_kernels():
    from tests.test_gpu_attention_plan import BALANCED
    reached = set()
    for B, n_list, Hq, Hkv, Dh, L_list in BALANCED:
        p = P.attention_plan(B, (max(n_list) + 63) // 64 * 64, Hq, Hkv, Dh, max(L_list))
        assert p["balance"] and device_run(p, n_list, Hq // Hkv, L_list) < p["run_bound"], (p, n_list, L_list)
        reached.add((Dh, p["waves"]))
    assert reached == {(64, 4), (64, 8), (128, 4), (128, 8)}
