"""Scoring and selection of small problems in one kernel: scores against the oracle and lists of dfs_forward against the staged
calls bit for bit, at one block, at the largest row the rule takes for each r and d and one beyond (the two kernels).  Then what
the scores lose to fp32."""
import numpy as np
import pytest
import torch

from oracle import dfs_oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("d,r,M_v,heads", [(64, 1, 1, 3), (64, 1, 12, 2), (64, 1, 13, 2), (64, 2, 1, 1), (64, 2, 64, 2), (64, 2, 65, 2), (64, 4, 2, 2),
                                           (64, 4, 65, 2), (64, 4, 320, 1), (64, 4, 321, 1), (64, 8, 1, 2), (64, 8, 256, 1), (64, 8, 257, 1), (128, 1, 12, 2),
                                           (128, 1, 13, 2), (128, 2, 32, 2), (128, 2, 33, 2), (128, 4, 320, 1), (128, 4, 321, 1), (128, 4, 9, 2),
                                           (128, 8, 256, 1), (128, 8, 257, 1), (128, 8, 64, 2), (128, 8, 5, 1)])
def test_scores_and_lists(d, r, M_v, heads):
    N_v = M_v * 64 - (64 // r % 64 + 3 if M_v % 2 else 0) if M_v > 1 else 41     # odd counts: a ragged last block, without its last sub-block if r > 1
    H, W = next((n // w, w) for n in range(N_v, 0, -1) for w in range(512, 0, -1) if n % w == 0 and n // w <= 512)
    n_text = 70 if heads == 2 else 0
    g = P.Geom(1, H, W, n_text, heads, d, 64, 64 // r)
    s = P.dfs_geom_sizes(g)
    assert s.M_v == M_v
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M_v * d + r)
    q, k, v = (torch.randn(heads, s.N, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    q, k = q * 3, k * 3
    perm_pad, inv, _ = G.gpu_perm(g)
    qp, kp = (G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in (q, k))
    score = G.gpu_score(g, P.DFS_BF16, qp, kp)
    # the bound of the scores everywhere: fp32 contraction, exponentials and sums of at most r x r probabilities
    want = O.block_score(qp[:1].float().cpu().numpy().astype(np.float64), kp[:1].float().cpu().numpy().astype(np.float64), s.N_v, 64, 64 // r)
    assert np.abs(score[0].cpu().numpy() - want.reshape(M_v, M_v)).max() <= 1e-5 * r
    i32 = dict(dtype=torch.int32, device="cuda")
    for mode, sparsity, mass in ((P.DFS_SELECT_TOPK, 0.7, 0.0), (P.DFS_SELECT_MASS_ROW, 0.95, 0.8)):
        K_max = s.M if mode != P.DFS_SELECT_TOPK else P.dfs_keep_count(sparsity, s.M_v) + s.M_x
        mask = torch.full((heads, s.M, s.M), 9, dtype=torch.uint8, device="cuda")
        st = P.MaskState(torch.full((heads, s.M, K_max), -1, **i32), torch.full((heads, s.M), -1, **i32), mask, torch.full((heads,), -1, **i32), K_max)
        P.dfs_forward(g, P.DFS_BF16, q, k, v, perm_pad, inv, True, mode, sparsity, mass, st, d ** -0.5, torch.empty_like(q),
                      G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16)))
        ref = G.gpu_select(g, score, mode, sparsity, mass, K_max=K_max)
        for name in ("kv_idx", "kv_cnt", "mask", "k_head"):
            assert torch.equal(getattr(st, name), getattr(ref, name)), (name, mode)


@pytest.mark.parametrize("d,B,r,M_v", [(64, 64, 8, 86), (128, 64, 8, 86), (128, 128, 4, 100), (64, 128, 4, 138)])
def test_scores_are_as_accurate_as_their_parts(d, B, r, M_v):
    """Rows of evenly spread scores over 400 to 700 key sub-blocks, whose log-sum-exp lies between 8 and 16: rounded to fp32 there it
    alone is off by 2^-21 and less, 2.8e-7 to 3.3e-7 of the scores in 2-norm on these inputs.  The block logarithms, of magnitude
    four and less, their logarithm, exponential and the sum's reciprocal are each good to 2^-23 and less: 2^-22 in all in 2-norm."""
    g = P.Geom(1, M_v, B, 0, 4, d, B, B // r)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M_v)
    q, k = (torch.randn(4, M_v * B, d, generator=gen, device="cuda").bfloat16() for _ in range(2))
    q_hat, k_hat = (x.double().reshape(4, M_v * r, B // r, d).mean(2) for x in (q, k))
    probs = torch.softmax(q_hat @ k_hat.transpose(1, 2).contiguous() / d ** 0.5, -1)
    want = probs.reshape(4, M_v, r, M_v, r).sum((2, 4))
    err = float((G.gpu_score(g, P.DFS_BF16, q, k).double() - want).norm() / want.norm())
    print(f"d={d} r={r} M_v={M_v}: {err:.2e}", flush=True)
    assert err <= 2.0 ** -22


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("r", [1, 2, 4, 8])
def test_two_work_groups_a_cu(d, r):
    g = P.Geom(1, 12, 64, 0, 2, d, 64, 64 // r)
    s = P.dfs_geom_sizes(g)
    q = torch.zeros(2, s.N_pad, d, dtype=torch.bfloat16, device="cuda")
    score = torch.empty(2, s.M_v, s.M_v, device="cuda")
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_BLOCK_SCORE))
    assert G.resident_of(lambda: P.dfs_block_score(g, P.DFS_BF16, q, q, score, ws))[f"score_small_kernel<{d}, {r}>"] >= 2
