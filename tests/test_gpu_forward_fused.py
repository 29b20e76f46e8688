"""dfs_forward against the staged calls, bit for bit, at the sub-block sizes that make the pooling kernel's row groups in flight one
short pass, whole passes and several, with ragged last sub-blocks and text: with an output of its own (bf16 tensors: the attention gathers
K and V) and with one over the keys or the values, where a refresh step's pooling reorders both on the way before the first row is
written, and a reuse step's gather does (fp32 tensors: always)."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("dtype", [P.DFS_BF16, P.DFS_F32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Bs,W,n_text", [(64, 8, 75, 3), (64, 16, 64, 0), (128, 16, 90, 129), (128, 32, 77, 40), (64, 64, 33, 0), (128, 128, 101, 7)])
def test_forward_equals_staged_calls(dtype, d, B, Bs, W, n_text):
    g = P.Geom(2, 5, W, n_text, 2, d, B, Bs)
    s = P.dfs_geom_sizes(g)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    td = torch.bfloat16 if dtype == P.DFS_BF16 else torch.float32
    q, k, v = (torch.randn(2, s.N, d, generator=gen, device="cuda").to(td) for _ in range(3))
    perm_pad, inv, _ = G.gpu_perm(g)
    K_max = P.dfs_keep_count(0.5, s.M_v) + s.M_x
    i32 = dict(dtype=torch.int32, device="cuda")
    st = P.MaskState(torch.zeros((2, s.M, K_max), **i32), torch.zeros((2, s.M), **i32), None, None, K_max)
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16 if dtype == P.DFS_BF16 else P.DFS_WS_FORWARD))
    ws.fill_(255)
    kp, vp = (G.gpu_permute(g, dtype, x, perm_pad) for x in (k, v))
    qp = G.gpu_permute(g, dtype, q, perm_pad)
    st2 = G.gpu_select(g, G.gpu_score(g, dtype, qp, kp), P.DFS_SELECT_TOPK, 0.5)
    want = G.gpu_unperm(g, dtype, G.gpu_attn(g, dtype, qp, kp, vp, st2, want_lse=False)[0], inv)
    for refresh in (True, False):
        for over in (None, "k", "v"):
            x = [q, k, v]
            o = torch.full_like(q, float("nan"))
            if over:
                x["qkv".index(over)] = o
                o.copy_(k if over == "k" else v)
            kernels = G.kernels_of(lambda: P.dfs_forward(g, dtype, *x, perm_pad, inv, refresh, P.DFS_SELECT_TOPK, 0.5, 0.0, st, 1.0 / math.sqrt(d), o, ws))
            assert not any("gather_rows" in name for name in kernels) or not refresh
            assert dtype == P.DFS_F32 or kernels[-1].endswith(", 0>" if over else ", 1>")        # from the reordered copies, or gathered
            P.dfs_forward(g, dtype, *x, perm_pad, inv, refresh, P.DFS_SELECT_TOPK, 0.5, 0.0, st, 1.0 / math.sqrt(d), o, ws)
            assert torch.equal(st.kv_cnt, st2.kv_cnt)
            assert torch.equal(o.view(torch.uint8), want.view(torch.uint8)), (refresh, over)
