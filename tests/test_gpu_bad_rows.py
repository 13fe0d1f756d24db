"""Rows that cannot be normalised are reported wherever the NaN lies: also where the lane that reads it sees
no other logit (the ragged end of a row, a masked vocabulary), in every call that scans rows."""
import numpy as np
import pytest

from tests import harness as H
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu
PLACES = 6


def place_nan(row, place, block):
    """row: [V] float32; block: logits a workgroup holds at a time (a lane's vectors of the next block lie one block on)."""
    V = row.shape[0]
    if place == 0:                  # the last token, alone in its vector where the vocabulary is ragged
        row[V - 1] = np.nan
    elif place == 1:                # a masked vocabulary, the NaN behind the only token left
        row[:] = -np.inf
        row[3], row[V - 1] = 1.0, np.nan
    elif place == 2:                # ... in front of it, in the same lane a block earlier
        row[:] = -np.inf
        row[1000], row[1000 + block] = np.nan, 1.0
    elif place == 3:                # ... in another lane of the same block
        row[:] = -np.inf
        row[5], row[2000] = 1.0, np.nan
    elif place == 4:                # a whole block
        row[:block] = np.nan
    else:                           # nothing but -inf and NaN
        row[:] = -np.inf
        row[V // 2] = np.nan


def rows_with_nans(dtype, V, rows, bad_row):
    """[1 + PLACES][rows][V]: sequence 0 is clean, sequence 1 + p has place p in row `bad_row`."""
    rng = np.random.default_rng(V + rows)
    x = rng.standard_normal((1 + PLACES, rows, V), dtype=np.float32) * 3
    block = 4096 if dtype == "f32" else 8192
    for p in range(PLACES):
        place_nan(x[1 + p, bad_row], p, block)
    return x


def on_device(x, dtype):
    import torch
    B, R, V = x.shape
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    dev = torch.full((B, R, (V + 7) // 8 * 8), 100.0, dtype=dt, device="cuda")   # what lies behind a row has no effect
    dev[:, :, :V] = torch.from_numpy(x).to(dt).cuda()
    return dev[:, :, :V]


# runs of one block (few rows), of two and of five
@pytest.mark.parametrize("dtype,V,N", [("bf16", 50257, 6), ("bf16", 50001, 100), ("bf16", 50001, 256), ("f32", 20001, 6), ("f32", 20001, 256)])
def test_target_argmax_reports_every_nan(dtype, V, N):
    import torch
    import paper_2601_07353_amd as T
    print("case", dtype, V, N, flush=True)
    B = 1 + PLACES
    logits = on_device(rows_with_nans(dtype, V, N, N - 2), dtype)
    st = T.TreeState(B, N)
    st.n_nodes.fill_(N)
    ws = T.make_verify_workspace(B, st.N_pad, V, T.TALON_DTYPE_F32 if dtype == "f32" else T.TALON_DTYPE_BF16)
    tok = torch.zeros(B, st.N_pad, dtype=torch.int32, device="cuda")
    status = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    T.talon_target_argmax(logits, st, tok, None, status, ws)
    assert status.tolist() == [0] + [T.TALON_STATUS_BAD_ROW] * PLACES
    np.testing.assert_array_equal(tok[0, :N].cpu().numpy(), logits[0].float().argmax(-1).cpu().numpy())


@pytest.mark.parametrize("how", ["ahead", "layered", "tree", "fused", "split", "literal", "literal-ahead", "literal-ahead-wide"])
@pytest.mark.parametrize("dtype,V", [("bf16", 50257), ("f32", 20001)])
def test_expansion_reports_every_nan(dtype, V, how):
    import torch
    import paper_2601_07353_amd as T
    print("case", dtype, V, how, flush=True)
    B = 1 + PLACES
    cfg = small(name="nan-rows", V=V, logits_dtype=dtype, K=4, N=100 if how == "literal-ahead-wide" else 24, Dmax=6, B=B)
    logits = on_device(rows_with_nans(dtype, V, cfg.N_pad, 0), dtype)
    if how.startswith("literal"):
        st = T.TreeState(B, cfg.N)
        ws = T.make_literal_workspace(B, st.N_pad, V, T.TALON_DTYPE_F32 if dtype == "f32" else T.TALON_DTYPE_BF16)
        T.talon_tree_init(st, torch.arange(B, dtype=torch.int32, device="cuda"))
        T.talon_expand_literal(logits, st, 1 if how == "literal" else cfg.Dmax, cfg.mu, cfg.K, 1, cfg.Dmax, ws)
    else:
        st, _, _, _ = H.run_gpu_expand(cfg, logits, layerwise=False if how == "ahead" else how)
    status, n = st.status.tolist(), st.n_nodes.tolist()
    assert not status[0] & T.TALON_STATUS_BAD_ROW and n[0] > 1
    for p in range(PLACES):
        assert status[1 + p] & T.TALON_STATUS_BAD_ROW and n[1 + p] == 1, (p, status, n)


@pytest.mark.parametrize("dtype,V,N", [("bf16", 50257, 6), ("bf16", 17, 6), ("f32", 20001, 256)])
def test_target_argmax_leaves_no_stale_token_in_a_row_of_infinities(dtype, V, N):
    """Nothing but -inf: reported, and the token is the first one, not what the buffer held before."""
    import torch
    import paper_2601_07353_amd as T
    print("case", dtype, V, N, flush=True)
    x = np.random.default_rng(V).standard_normal((2, N, V), dtype=np.float32)
    x[1, 2:] = -np.inf
    logits = on_device(x, dtype)
    st = T.TreeState(2, N)
    st.n_nodes.fill_(N)
    ws = T.make_verify_workspace(2, st.N_pad, V, T.TALON_DTYPE_F32 if dtype == "f32" else T.TALON_DTYPE_BF16)
    tok = torch.full((2, st.N_pad), -7, dtype=torch.int32, device="cuda")
    prob = torch.full((2, st.N_pad), -7.0, device="cuda")
    status = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    T.talon_target_argmax(logits, st, tok, prob, status, ws)
    assert status.tolist() == [0, T.TALON_STATUS_BAD_ROW]
    want = logits.float().argmax(-1).cpu().numpy()
    want[1, 2:] = 0
    np.testing.assert_array_equal(tok[:, :N].cpu().numpy(), want)
    assert torch.isnan(prob[1, 2:N]).all() and not torch.isnan(prob[0]).any()


@pytest.mark.parametrize("dtype,V,N", [("bf16", 50257, 24), ("f32", 20001, 24), ("bf16", 50257, 256)])
def test_a_mask_of_the_lowest_value_is_as_good_as_infinities(dtype, V, N):
    """Rows of which all but a few tokens are masked, with -inf in sequence 0 and with the type's lowest value in
    sequence 1 (sequence 2: the lowest value behind the first 8192 tokens): the same tokens, none of them bad."""
    import torch
    import paper_2601_07353_amd as T
    print("case", dtype, V, N, flush=True)
    cfg = small(name="masked", V=V, logits_dtype=dtype, K=4, N=N, Dmax=6, B=4)
    P = cfg.N_pad
    low = float(torch.finfo(torch.float32 if dtype == "f32" else torch.bfloat16).min)
    rng = np.random.default_rng(V)
    x = np.empty((4, P, V), dtype=np.float32)
    x[0] = rng.standard_normal((P, V), dtype=np.float32) * 3
    few = rng.random((P, V)) < 40.0 / V
    few[:, rng.integers(0, V, 8)] = True      # (no row without a token)
    x[2] = x[0]
    x[2, :, 8192:] = low
    x[3] = np.where(np.arange(V) < 8192, x[0], -np.inf)
    x[1] = np.where(few, x[0], low)
    x[0] = np.where(few, x[0], -np.inf)
    logits = on_device(x, dtype)
    same = lambda a, b, *ts: [np.testing.assert_array_equal(t[a].cpu().numpy(), t[b].cpu().numpy()) for t in ts]
    st = T.TreeState(4, N)
    st.n_nodes.fill_(N)
    ws = T.make_verify_workspace(4, P, V, T.TALON_DTYPE_F32 if dtype == "f32" else T.TALON_DTYPE_BF16)
    tok, status = torch.zeros(4, P, dtype=torch.int32, device="cuda"), torch.full((4,), -1, dtype=torch.int32, device="cuda")
    prob = torch.zeros(4, P, device="cuda")
    T.talon_target_argmax(logits, st, tok, prob, status, ws)
    assert status.tolist() == [0] * 4
    same(0, 1, tok, prob)
    same(2, 3, tok, prob)
    for how in (False, "layered", "fused", "split"):
        st, cand, _, _ = H.run_gpu_expand(cfg, logits, layerwise=how)
        assert not any(s & T.TALON_STATUS_BAD_ROW for s in st.status.tolist())
        for a, b in ((0, 1), (2, 3)):
            n = int(st.n_nodes[a])
            assert n == int(st.n_nodes[b]) > 1
            same(a, b, st.token[:, 1:n], st.parent[:, :n], st.prob[:, :n], st.logp[:, :n])
