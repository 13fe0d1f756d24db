"""csrc/marshal.cpp: what reaches the C ABI and what is refused on the way (no GPU needed: every call here ends
in an argument check of the library or of the marshalling)."""
import ctypes

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
