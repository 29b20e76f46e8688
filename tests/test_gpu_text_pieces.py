"""Text rows of problems whose work-groups all start at once, dealt in pieces of five eighths of a video row where that pays: lists at which the pieces are
the least, a little more, and leave a last one of a single block, and at the rules' limits, by the number of work-groups; against float64 on the same tensors."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("d,B,H,W,n_text,heads,kept,piece", [
    (64, 64, 32, 42, 30, 4, 10, 8), (64, 128, 64, 80, 200, 3, 10, 8),      # five eighths of 11 and 12 blocks are 6 and 7: the least piece instead
    (64, 64, 32, 80, 77, 3, 13, 9), (128, 64, 32, 80, 130, 2, 17, 12), (64, 128, 64, 80, 200, 3, 14, 10), (128, 128, 64, 81, 128, 3, 18, 11),
    (128, 128, 64, 81, 400, 3, 14, 11), (64, 64, 32, 80, 300, 2, 13, 11),  # the last piece is one block
    (64, 64, 32, 80, 77, 3, 10, 12), (64, 64, 32, 80, 77, 3, 11, 13), (128, 64, 32, 80, 77, 3, 10, 8),     # two pieces more for four and five blocks
    (64, 128, 64, 81, 30, 12, 19, 12),                     # 528 work-groups -> 540
    (64, 64, 45, 57, 1, 16, 15, 10), (64, 64, 45, 57, 1, 17, 15, 16),      # 736 work-groups with them, 782
    (64, 64, 32, 42, 259, 15, 6, 11), (64, 64, 24, 40, 259, 20, 5, 10),    # 75 work-groups more, 500 -> 600: one wave group instead of two
    (128, 128, 64, 58, 256, 7, 13, 15), (128, 128, 64, 58, 256, 6, 13, 9)])      # 245 -> 259, a second one on some CUs; 210 -> 222
def test_text_rows_in_short_pieces(d, B, H, W, n_text, heads, kept, piece):
    g = P.Geom(1, H, W, n_text, heads, d, B, B // 4)
    s = P.dfs_geom_sizes(g)
    sparsity = 1 - kept / s.M_v
    K_max = kept + s.M_x
    assert P.dfs_keep_count(sparsity, s.M_v) == kept and 2 * K_max <= s.M and s.M >= 16 and heads * s.M <= (512 if B == 128 else 1024)
    pieces = -(-s.M // piece)
    assert piece in (max(8, K_max * 5 // 8), max(8, K_max))
    probe = torch.zeros(3, dtype=torch.int64, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + kept)
    q, k, v = (torch.randn(heads, s.N, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    perm_pad, inv, _ = G.gpu_perm(g)
    i32 = dict(dtype=torch.int32, device="cuda")
    st = P.MaskState(torch.zeros((heads, s.M, K_max), **i32), torch.zeros((heads, s.M), **i32), None, None, K_max)
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16))
    outs = []
    for refresh in (True, False, False):
        out = torch.full_like(q, float("nan"))
        P.dfs_attn_clock_probe(probe.zero_())
        try:
            P.dfs_forward(g, P.DFS_BF16, q, k, v, perm_pad, inv, refresh, P.DFS_SELECT_TOPK, sparsity, 0.0, st, d ** -0.5, out, ws)
            torch.cuda.synchronize()
        finally:
            P.dfs_attn_clock_probe(None)
        assert int(probe[2]) == heads * (s.M_v + s.M_x * pieces)
        outs.append(out)
    assert torch.isfinite(outs[0].float()).all() and all(torch.equal(outs[0], o) for o in outs[1:])
    qf, kf, vf = (x.double().cpu() for x in (q[:, s.N_v:], k, v))
    want = torch.softmax(qf @ kf.transpose(1, 2) * d ** -0.5, -1) @ vf
    got = outs[0][:, s.N_v:].double().cpu()
    # weights and result are rounded to bf16, 1.9e-3 of the result in 2-norm: four times that, the suite's bound
    assert float((got - want).norm() / want.norm()) <= 7.5e-3
