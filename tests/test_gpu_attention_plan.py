"""Split-KV plans of tree attention: batches of unequal prefixes (the run length is worked out on the
device), and calls whose workspace was sized for another prefix."""
import numpy as np
import pytest

from tests import harness as H
from tests.test_gpu_parity import attention_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n_list,Hq,Hkv,Dh,L_list", [
    (3, [40, 3, 64], 8, 2, 128, [3000, 0, 70]),                       # one long prefix: the others take one run
    (2, [100, 1], 4, 2, 64, [1500, 0]),                               # a lone root without a prefix beside a full tree
    (70, [1 + (7 * i) % 60 for i in range(70)], 4, 4, 64, [(37 * i) % 1100 for i in range(70)]),   # two sequences per lane
    (5, [90, 30, 128, 70, 1], 24, 8, 64, [1100, 64, 65, 700, 4500]),  # more runs for the long ones than full lengths would get
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
