"""csrc/marshal.cpp: what reaches the C ABI and what is refused on the way (no GPU needed: every call here ends
in an argument check of the library or of the marshalling)."""
import ctypes
from decimal import Decimal
from fractions import Fraction

import numpy as np
import pytest
import torch

import paper_2601_07353_amd as T
from paper_2601_07353_amd import binding


@pytest.fixture(scope="module")
def buffers():
    T.load_library()
    st = T.TreeState(2, 30, device="cpu")
    cand = T.Candidates(2, 64, 4, device="cpu")
    return st, cand, torch.zeros(1 << 22, dtype=torch.uint8), torch.zeros(2, 64, 1000, dtype=torch.bfloat16)


def refused(code, text, call):
    with pytest.raises(T.TalonError) as e:
        call()
    assert e.value.code == code and text in str(e.value), str(e.value)


def test_loop_calls_go_through_the_marshalling_module():
    T.load_library()
    assert binding._native.__name__ == "_talon_marshal"


def test_values_arrive_where_they_belong(buffers):
    """The library names the argument it refuses, with its value."""
    st, cand, ws, logits = buffers
    how = (0.03, 5, 1, 6)
    layer = lambda k=4, how=how, lg=logits, w=ws, **kw: T.talon_expand_select_layer(lg, st, k, *how, cand, w, stream=0, **kw)
    refused(T.TALON_ERR_INVALID_ARG, "k=65", lambda: layer(k=65))
    refused(T.TALON_ERR_INVALID_ARG, "mu=2", lambda: layer(how=(2, 5, 1, 6)))
    refused(T.TALON_ERR_INVALID_ARG, "K_init=0", lambda: layer(how=(0.03, 0, 1, 6)))
    refused(T.TALON_ERR_INVALID_ARG, "init_layers=-1", lambda: layer(how=(0.03, 5, -1, 6)))
    refused(T.TALON_ERR_INVALID_ARG, "max_depth=0", lambda: layer(how=(0.03, 5, 1, 0)))
    refused(T.TALON_ERR_INVALID_ARG, "row_mode=3", lambda: layer(row_mode=3))
    refused(T.TALON_ERR_INVALID_ARG, "row_stride=1000", lambda: layer(vocab=1001))
    refused(T.TALON_ERR_WORKSPACE, "workspace of 512 bytes", lambda: layer(w=ws[:512]))
    refused(T.TALON_ERR_INVALID_ARG, "k=0", lambda: T.talon_expand_layer(logits, st, 0, cand, ws, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "mu=-1", lambda: T.talon_select_budget(st, 4, cand, -1.0, 5, 1, 6, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "root_token is NULL", lambda: T.talon_tree_init(st, None, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "max_depth=0", lambda: T.talon_build_tree(st.token, logits, st, 4, 0.03, 5, 1, 0, cand, ws, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "K_init=0", lambda: T.talon_expand_literal(logits, st, 3, 0.03, 0, 1, 6, ws, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "mask is NULL", lambda: T.talon_build_tree_mask(st, None, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "scan_status is NULL", lambda: T.talon_target_argmax(logits, st, cand.token, None, None, ws, stream=0))
    kv = torch.zeros(2, 64, 2, 64, dtype=torch.bfloat16)
    n = torch.zeros(2, dtype=torch.int32)
    refused(T.TALON_ERR_UNSUPPORTED, "Hq/Hkv=17", lambda: T.talon_tree_attention(
        torch.zeros(2, 64, 34, 64, dtype=torch.bfloat16), kv, kv, kv, kv, st.token, n, n, 64, kv, stream=0))
    odd = torch.zeros(2, 64, 2, 60, dtype=torch.bfloat16)
    refused(T.TALON_ERR_INVALID_ARG, "Hkv=2, Dh=60", lambda: T.talon_compact_kv(odd, odd, n, n, n, n, kv, kv, stream=0))


def test_what_is_refused_before_the_library(buffers):
    st, cand, ws, logits = buffers
    layer = lambda lg, k=4, mu=0.03: T.talon_expand_select_layer(lg, st, k, mu, 5, 1, 6, cand, ws, stream=0)
    refused(T.TALON_ERR_UNSUPPORTED, "torch.float16", lambda: layer(logits.half()))
    refused(T.TALON_ERR_INVALID_ARG, "contiguous rows", lambda: layer(logits[:, :, ::2]))
    refused(T.TALON_ERR_INVALID_ARG, "contiguous rows", lambda: layer(logits[0]))
    for bad in (lambda: layer(logits, k=4.0), lambda: layer(logits, k="4"), lambda: layer(logits, k=None), lambda: layer(logits, mu="x"),
                lambda: T.talon_expand_select_layer(logits, st, 4, 0.03, 5, 1, 6, cand, ws, layer=None, stream=0)):
        with pytest.raises(TypeError):
            bad()
    with pytest.raises(AttributeError):
        T.talon_expand_select_layer(logits, st, 4, 0.03, 5, 1, 6, object(), ws, stream=0)
    with pytest.raises(TypeError):
        binding._native.tree_init(st.c, st.token)
    with pytest.raises(TypeError):
        binding._native.tree_init(ctypes.c_int(1), st.token, 0)
    kv = torch.zeros(2, 64, 2, 64, dtype=torch.bfloat16)
    n = torch.zeros(2, dtype=torch.int32)
    refused(T.TALON_ERR_INVALID_ARG, "must be contiguous", lambda: T.talon_tree_attention(
        kv.transpose(1, 2), kv, kv, kv, kv, st.token, n, n, 64, kv, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "share strides", lambda: T.talon_tree_attention(
        kv, kv, torch.zeros(2, 64, 2, 128, dtype=torch.bfloat16)[..., :64], kv, kv, st.token, n, n, 64, kv, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "share strides", lambda: T.talon_compact_kv(kv, kv, n, n, n, n, kv, kv.transpose(0, 2), stream=0))


class _Index:
    def __index__(self):
        return 65


class _Parameter:
    _as_parameter_ = ctypes.c_int32(65)


@pytest.mark.parametrize("k", [np.int64(65), np.int32(65), np.uint8(65), torch.tensor(65), torch.tensor([65], dtype=torch.int32),
                               ctypes.c_int32(65), _Index(), _Parameter()], ids=lambda v: type(v).__name__)
def test_whole_numbers_of_every_kind_arrive(buffers, k):
    """What a foreign function's integer argument takes, the marshalled calls take in every integer place."""
    st, cand, ws, logits = buffers
    refused(T.TALON_ERR_INVALID_ARG, "k=65", lambda: T.talon_expand_select_layer(logits, st, k, 0.03, 5, 1, 6, cand, ws, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "k=65", lambda: T.talon_expand_layer(logits, st, k, cand, ws, stream=0, vocab=None))
    refused(T.TALON_ERR_INVALID_ARG, "k=65", lambda: T.talon_select_budget(st, k, cand, 0.03, 5, 1, 6, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "row_mode=65", lambda: T.talon_expand_tree(logits, st, 4, 0.03, 5, 1, 6, cand, ws, row_mode=k, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "K_init=0", lambda: T.talon_build_tree(
        st.token, logits, st, 4, 0.03, 0, k, k, cand, ws, stream=0, vocab=k))
    refused(T.TALON_ERR_INVALID_ARG, "K_init=0", lambda: T.talon_expand_literal(logits, st, k, 0.03, 0, k, k, ws, stream=0, vocab=k))
    refused(T.TALON_ERR_INVALID_ARG, "scan_status is NULL", lambda: T.talon_target_argmax(
        logits, st, cand.token, None, None, ws, vocab=k, stream=0))
    kv = torch.zeros(2, 64, 2, 64, dtype=torch.bfloat16)
    n = torch.zeros(2, dtype=torch.int32)
    refused(T.TALON_ERR_UNSUPPORTED, "Hq/Hkv=17", lambda: T.talon_tree_attention(
        torch.zeros(2, 64, 34, 64, dtype=torch.bfloat16), kv, kv, kv, kv, st.token, n, n, k, kv, stream=0))


@pytest.mark.parametrize("mu", [np.float32(2), np.float64(2), np.int64(2), torch.tensor(2.0), Decimal(2), Fraction(2), ctypes.c_float(2)],
                         ids=lambda v: type(v).__name__)
def test_numbers_of_every_kind_arrive(buffers, mu):
    st, cand, ws, logits = buffers
    refused(T.TALON_ERR_INVALID_ARG, "mu=2", lambda: T.talon_expand_select_layer(logits, st, 4, mu, 5, 1, 6, cand, ws, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "mu=2", lambda: T.talon_select_budget(st, 4, cand, mu, 5, 1, 6, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "mu=2", lambda: T.talon_expand_literal(logits, st, 3, mu, 5, 1, 6, ws, stream=0))
    kv = torch.zeros(2, 64, 2, 64, dtype=torch.bfloat16)
    n = torch.zeros(2, dtype=torch.int32)
    refused(T.TALON_ERR_UNSUPPORTED, "Hq/Hkv=17", lambda: T.talon_tree_attention(
        torch.zeros(2, 64, 34, 64, dtype=torch.bfloat16), kv, kv, kv, kv, st.token, n, n, 64, kv, scale=mu, stream=0))


def test_heads_of_tree_keys_come_from_their_third_dimension(buffers):
    st, _, _, _ = buffers
    kv = torch.zeros(2, 64, 2, 64, dtype=torch.bfloat16)
    n = torch.zeros(2, dtype=torch.int32)
    q = torch.zeros(2, 64, 34, 64, dtype=torch.bfloat16)
    for keys in (kv.view(2, 64, 2, 8, 8), kv.view(2, 64, 2, 64)):
        refused(T.TALON_ERR_UNSUPPORTED, "Hq/Hkv=17", lambda: T.talon_tree_attention(q, kv, kv, keys, kv, st.token, n, n, 64, kv, stream=0))
    refused(T.TALON_ERR_INVALID_ARG, "k_tree must be", lambda: T.talon_tree_attention(
        q, kv, kv, torch.zeros(2, 64), kv, st.token, n, n, 64, kv, stream=0))
