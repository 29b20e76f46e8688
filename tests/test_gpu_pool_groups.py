"""Pooling with a wave for four sub-blocks (pool_read_kernel): scores bit for bit those of the kernel that pools one a wave, which a problem of
few heads takes.  Ragged last sub-blocks and groups, every sub-block size, text, orders with entries that are none, both layouts of the centroids."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("H,W,n_text,heads,d,B,Bs", [
    (1, 5, 0, 400, 64, 64, 8), (7, 13, 9, 200, 64, 64, 16), (20, 67, 0, 40, 64, 64, 32), (20, 67, 70, 40, 128, 128, 32), (33, 61, 5, 13, 128, 64, 16),
    (19, 27, 0, 30, 128, 64, 8), (150, 278, 0, 3, 64, 128, 32), (150, 277, 1, 2, 128, 128, 16)])
def test_same_scores(H, W, n_text, heads, d, B, Bs):
    g, one = (P.Geom(1, H, W, n_text, h, d, B, Bs) for h in (heads, 1))
    s = P.dfs_geom_sizes(g)
    assert heads * ((s.M_s + 3) // 4) >= 384
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    q, k, v = (torch.randn(heads, s.N, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    q[1], k[-1] = q[1] * 2.0 ** 60, k[-1] * 2.0 ** -60         # scales far from one
    perm_pad, inv, _ = G.gpu_perm(g)
    if n_text:
        perm_pad[::17] = torch.tensor([-1, s.N, 2 ** 31 - 1], dtype=torch.int32, device="cuda").repeat(s.N_pad)[:perm_pad[::17].numel()]
    qp, kp = (G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in (q, k))
    assert G.kernels_of(lambda: G.gpu_score(g, P.DFS_BF16, qp, kp))[0] == f"pool_read_kernel<{d}>"
    score = G.gpu_score(g, P.DFS_BF16, qp, kp)
    few = min(heads, 3) if (s.M_s + 3) // 4 < 384 else 0              # else one head alone is pooled in the same way
    for h in list(range(few)) + ([heads - 1] if few else []):
        assert G.kernels_of(lambda: G.gpu_score(one, P.DFS_BF16, qp[h:h + 1], kp[h:h + 1]))[0] == f"pool_kernel<1, {d}>"
        assert torch.equal(score[h:h + 1], G.gpu_score(one, P.DFS_BF16, qp[h:h + 1].contiguous(), kp[h:h + 1].contiguous()))
    # from the tensors in source order (both of them, as dfs_forward does): the lists of those scores
    K_max = P.dfs_keep_count(0.6, s.M_v) + s.M_x
    want = G.gpu_select(g, score, P.DFS_SELECT_TOPK, 0.6, K_max=K_max)
    i32 = dict(dtype=torch.int32, device="cuda")
    st = P.MaskState(torch.zeros((heads, s.M, K_max), **i32), torch.zeros((heads, s.M), **i32), torch.zeros((heads, s.M, s.M), dtype=torch.uint8, device="cuda"), None, K_max)
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16))
    step = lambda: P.dfs_forward(g, P.DFS_BF16, q, k, v, perm_pad, inv, True, P.DFS_SELECT_TOPK, 0.6, 0.0, st, d ** -0.5, torch.empty_like(q), ws)  # noqa: E731
    assert G.kernels_of(step)[0] == f"pool_read_kernel<{d}>"
    step()
    assert torch.equal(st.mask, want.mask) and torch.equal(st.kv_cnt, want.kv_cnt)
