"""Split-KV plans of tree attention: batches of unequal prefixes (with the balancing, the run length is
worked out on the device; without it, runs beyond the end of a sequence are empty), and calls whose
workspace was sized for another prefix."""
import numpy as np
import pytest

from tests import harness as H
from tests.test_gpu_parity import attention_case

pytestmark = pytest.mark.gpu


# Batches that balance, with runs shorter than full-length prefixes would get: one for each of the four
# kernels (heads of 64 and 128, 4 and 8 wavefronts).
BALANCED = [
    (3, [115, 10, 4], 32, 4, 128, [4, 299, 2471]),                    # 128, 8 wavefronts
    (5, [129, 42, 49, 38, 61], 12, 4, 128, [37, 603, 707, 2363, 196]),   # 128, 4
    (3, [3, 104, 6], 32, 4, 64, [2596, 43, 217]),                     # 64, 8
    (5, [130, 19, 17, 24, 14], 12, 4, 64, [70, 244, 2061, 473, 1487]),   # 64, 4
]


@pytest.mark.parametrize("B,n_list,Hq,Hkv,Dh,L_list", BALANCED)
def test_unequal_prefixes_that_share_the_grid(B, n_list, Hq, Hkv, Dh, L_list):
    attention_case(B, n_list, Hq, Hkv, Dh, L_list, seed=12, keys_atol=H.ATTN_KEYS_ATOL_CUT)


@pytest.mark.parametrize("B,n_list,Hq,Hkv,Dh,L_list", [
    (3, [40, 3, 64], 8, 2, 128, [3000, 0, 70]),                       # one long prefix: the others take one run
    (2, [100, 1], 4, 2, 64, [1500, 0]),                               # a lone root without a prefix beside a full tree
    (70, [1 + (7 * i) % 60 for i in range(70)], 4, 4, 64, [(37 * i) % 1100 for i in range(70)]),   # two sequences per lane
    (5, [90, 30, 128, 70, 1], 24, 8, 64, [1100, 64, 65, 700, 4500]),  # more runs for the long ones than full lengths would get
    (1, [30], 2, 1, 128, [33000]),                                    # more than 64 runs
])
def test_unequal_prefixes(B, n_list, Hq, Hkv, Dh, L_list):
    attention_case(B, n_list, Hq, Hkv, Dh, L_list, seed=11)


def test_every_accepted_workspace_gives_the_same_attention():
    """A smaller workspace than the query returns is refused or served with fewer splits.  Two plans round
    their softmax weights against different running maxima, so each is within the harness's bound of
    the exact value (2^-8 relative for the output, six standard deviations of the weights' rounding)
    and they are within twice that of each other."""
    import torch
    import paper_2601_07353_amd as T
    B, P, Hq, Hkv, Dh, L = 4, 64, 32, 8, 64, 6000
    g = torch.Generator().manual_seed(2)
    t = lambda *s: torch.randn(*s, generator=g).bfloat16().cuda()
    q, kt, vt, kp, vp = t(B, P, Hq, Dh), t(B, P, Hkv, Dh), t(B, P, Hkv, Dh), t(B, L, Hkv, Dh), t(B, L, Hkv, Dh)
    st = T.TreeState(B, 60)
    st.n_nodes.copy_(torch.tensor([60, 17, 0, 33], dtype=torch.int32))
    st.parent.zero_()
    st.parent[:, 0] = -1
    mask = torch.zeros(B, P, 1, dtype=torch.int64, device="cuda")
    T.talon_build_tree_mask(st, mask)
    plen = torch.tensor([L, 700, 5000, 2900], dtype=torch.int32, device="cuda")
    full = T.talon_tree_attention_workspace_bytes(B, P, Hq, Hkv, Dh, L)
    outs, refused = [], 0
    for nbytes in [full, full - 16, full // 2, full // 4, 256]:
        ws = torch.empty(nbytes // 16 * 16 + 4096, dtype=torch.uint8, device="cuda").fill_(0x7F)
        out = torch.zeros(B, P, Hq, Dh, dtype=torch.bfloat16, device="cuda")
        try:
            T.talon_tree_attention(q, kp, vp, kt, vt, mask, st.n_nodes, plen, L, out, workspace=ws[: nbytes // 16 * 16])
        except T.TalonError as e:
            assert e.code == T.TALON_ERR_WORKSPACE
            refused += 1
            continue
        torch.cuda.synchronize()
        assert bool((ws[nbytes // 16 * 16:] == 0x7F).all())     # nothing behind the workspace was touched
        outs.append(out.float().cpu().numpy())
        assert not out[2].any()                                  # a sequence without nodes
    assert len(outs) >= 2 and refused >= 1
    keys = plen.cpu().numpy().astype(np.float64)[:, None, None, None] + 1.0     # prefix and at least the node itself
    for o in outs[1:]:
        bound = 2.0 * (H.ATTN_OUT_RTOL * np.maximum(np.abs(o), np.abs(outs[0])) + H.ATTN_KEYS_ATOL / np.sqrt(keys))
        assert (np.abs(o - outs[0]) <= bound).all()


@pytest.mark.parametrize("n_list,Hq,Hkv,Dh,most,L_list", [
    ([150, 60, 60], 64, 16, 64, 793, [380, 440, 430]),                          # runs shortened to 5 tiles by the balancing
    ([256, 150, 150, 90, 256], 32, 4, 64, 2000, [2000, 900, 840, 880, 2000]),   # runs of 12 tiles, 18 where the chip is filled
])
def test_sequences_of_one_filling_run_are_rounded_once(n_list, Hq, Hkv, Dh, most, L_list):
    """A sequence that is one run in the plan that fills the chip stays one run in every other plan, and
    is rounded to bf16 once.  2-norm error against 64 bits: rounding a bf16 result costs
    sqrt(E[ulp^2] / 12) = 1.5e-3 of its root mean square, so do the softmax weights (independent of each
    other), 2.1-2.2e-3 together; a second rounding of partial results makes it 2.6-2.75e-3.  The bound
    lies between, over 10^5 elements and more of a sequence."""
    import torch
    import paper_2601_07353_amd as T
    B, N = len(n_list), max(n_list)
    P, G = (N + 63) // 64 * 64, Hq // Hkv
    g = torch.Generator(device="cuda").manual_seed(4)
    t = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    q, kt, vt, kp, vp = t(B, P, Hq, Dh), t(B, P, Hkv, Dh), t(B, P, Hkv, Dh), t(B, most, Hkv, Dh), t(B, most, Hkv, Dh)
    st = T.TreeState(B, N)
    st.n_nodes.copy_(torch.tensor(n_list, dtype=torch.int32))
    st.parent.zero_()
    st.parent[:, 0] = -1
    mask = torch.zeros(B, P, P // 64, dtype=torch.int64, device="cuda")
    T.talon_build_tree_mask(st, mask)
    plen = torch.tensor(L_list, dtype=torch.int32, device="cuda")
    ws = torch.empty(T.talon_tree_attention_workspace_bytes(B, P, Hq, Hkv, Dh, most), dtype=torch.uint8, device="cuda")
    out = torch.zeros(B, P, Hq, Dh, dtype=torch.bfloat16, device="cuda")
    T.talon_tree_attention(q, kp, vp, kt, vt, mask, st.n_nodes, plen, most, out, workspace=ws)
    again = torch.zeros_like(out)
    ws.fill_(0x7F)
    T.talon_tree_attention(q, kp, vp, kt, vt, mask, st.n_nodes, plen, most, again, workspace=ws)
    assert torch.equal(out, again)          # the same call on the same data repeats itself bit for bit
    single = 0
    for b in range(B):
        n, L = n_list[b], L_list[b]
        own = torch.eye(n, dtype=torch.bool, device="cuda")     # every node hangs below the root
        own[:, 0] = True
        err = ref = 0.0
        for h in range(Hkv):
            rows = q[b, :n, h * G:(h + 1) * G].double().reshape(n * G, Dh)
            K, V = (torch.cat([x[b, :L, h], y[b, :n, h]]).double() for x, y in ((kp, kt), (vp, vt)))
            s = rows @ K.t() / Dh ** 0.5
            s[:, L:].masked_fill_(~own.repeat_interleave(G, 0), float("-inf"))
            want = torch.softmax(s, -1) @ V
            err += float(((out[b, :n, h * G:(h + 1) * G].double().reshape(n * G, Dh) - want) ** 2).sum())
            ref += float((want ** 2).sum())
        if (L + 63) // 64 + (n + 63) // 64 <= {793: 8, 2000: 18}[most]:
            single += 1
            assert (err / ref) ** 0.5 < 2.4e-3, (b, (err / ref) ** 0.5)
        else:
            assert (err / ref) ** 0.5 < 3.0e-3, (b, (err / ref) ** 0.5)
    assert single >= 2
