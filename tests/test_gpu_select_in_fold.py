"""The selection inside dfs_forward, which forms a row's scores and selects in one kernel, against the staged calls bit for
bit (lists, counts, mask, keep counts), at block counts beside its groups of eight rows and of 64 columns, at the largest
row that fits its LDS and one beyond; and the keep count of the mass rules against the oracle on hand-made rows."""
import numpy as np
import pytest
import torch

from oracle import dfs_oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("mode,sparsity,mass", [(P.DFS_SELECT_TOPK, 0.7, 0.0), (P.DFS_SELECT_MASS_ROW, 0.9, 0.8), (P.DFS_SELECT_MASS_HEAD, 0.9, 0.8)])
@pytest.mark.parametrize("M_v,r,n_text", [(1, 1, 0), (7, 2, 65), (8, 4, 0), (9, 8, 1), (63, 4, 0), (65, 2, 130), (1728, 1, 0), (1729, 1, 64)])
def test_lists_equal_staged_calls(mode, sparsity, mass, M_v, r, n_text):
    # the first grid with that many blocks, its last one ragged if the count is odd
    H, W = next((n // w, w) for n in range(M_v * 64 - (17 if M_v % 2 else 0), 0, -1) for w in range(512, 0, -1) if n % w == 0 and n // w <= 512)
    g = P.Geom(1, H, W, n_text, 2, 64, 64, 64 // r)
    s = P.dfs_geom_sizes(g)
    assert s.M_v == M_v
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M_v)
    q, k, v = (torch.randn(2, s.N, 64, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    q, k = q * 3, k * 3
    perm_pad, inv, _ = G.gpu_perm(g)
    K_max = s.M if mode != P.DFS_SELECT_TOPK else P.dfs_keep_count(sparsity, s.M_v) + s.M_x
    i32 = dict(dtype=torch.int32, device="cuda")
    mask = torch.full((2, s.M, s.M), 9, dtype=torch.uint8, device="cuda")
    st = P.MaskState(torch.full((2, s.M, K_max), -1, **i32), torch.full((2, s.M), -1, **i32), mask, torch.full((2,), -1, **i32), K_max)
    o = torch.empty_like(q)
    P.dfs_forward(g, P.DFS_BF16, q, k, v, perm_pad, inv, True, mode, sparsity, mass, st, 0.125, o,
                  G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16)))
    score = G.gpu_score(g, P.DFS_BF16, *(G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in (q, k)))
    want = G.gpu_select(g, score, mode, sparsity, mass, K_max=K_max)
    for name in ("kv_idx", "kv_cnt", "mask", "k_head"):
        assert torch.equal(getattr(st, name), getattr(want, name)), name


@pytest.mark.parametrize("mass", [1e-9, 0.5, 0.9, 1.0])
@pytest.mark.parametrize("M_v", [2, 64, 130])
def test_mass_count_on_hand_made_rows(M_v, mass):
    g = P.Geom(1, 1, 64, 0, 1, 64, 64, 64) if M_v == 1 else P.Geom(1, M_v // 2, 128, 0, 1, 64, 64, 64)
    s = P.dfs_geom_sizes(g)
    assert s.M_v == M_v
    rng = np.random.default_rng(M_v)
    score = rng.random((1, M_v, M_v)).astype(np.float32)
    score[0, 0] = 0.25                                     # all equal
    score[0, 1] = np.where(np.arange(M_v) % 2, 0.0, -0.0)  # no mass at all
    if M_v > 2:
        score[0, 2] = 0.0; score[0, 2, 5] = 3e-8           # below the fixed point's step
        score[0, 3] = 2.0 ** -np.arange(M_v)
        score[0, 4] = -score[0, 4]; score[0, 4, -1] = 1.0
        score[0, 5, ::3] = 5000.0                          # beyond the clamp
        score[0, 6] = np.float32(0.1) + (np.arange(M_v) % 4).astype(np.float32) * np.float32(2.0 ** -27)      # keys apart in their last bits
    st = G.gpu_select(g, torch.from_numpy(score).cuda(), P.DFS_SELECT_MASS_ROW, 1.0, mass)
    want = [max(1, O.mass_keep_count(score[0, u].astype(np.float64), mass)) for u in range(M_v)]
    assert st.kv_cnt[0].cpu().tolist() == want
