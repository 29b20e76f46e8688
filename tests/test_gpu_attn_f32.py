"""fp32 attention where its split of a row's keys over eight waves can go wrong: fewer runs of 32 keys than waves, counts that
are no multiple of eight, ragged last blocks of 1, 31, 32 and 33 rows, empty and dense lists, and pad rows that hold NaN
(they must never be read into a result).  Against the oracle under the same lists; 1e-4 is the suite's bound for fp32."""
import numpy as np
import pytest
import torch

from oracle import dfs_oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,n_video,n_text", [(64, 1, 0), (64, 64, 0), (64, 97, 0), (64, 5 * 64 + 31, 33), (128, 160, 1), (128, 3 * 128 + 33, 130),
                                              (128, 9 * 128 + 32, 0)])
def test_f32_attention_edges(d, B, n_video, n_text):
    g = P.Geom(1, 1, n_video, n_text, 2, d, B, B // 4) if n_video <= 512 else P.Geom(1, n_video // 32, 32, n_text, 2, d, B, B // 4)
    s = P.dfs_geom_sizes(g)
    rng = np.random.default_rng(n_video + d)
    valid = G.gpu_perm(g)[2].cpu().numpy()
    q, k, v = (rng.standard_normal((2, s.N_pad, d)).astype(np.float32) for _ in range(3))
    pad = np.concatenate([np.arange(B) >= valid[b] for b in range(s.M)])
    clean = [x.astype(np.float64) for x in (q, k, v)]
    for x in (k, v):
        x[:, pad] = np.nan
    mask = np.zeros((2, s.M, s.M), dtype=np.uint8)
    for h in range(2):
        for u in range(s.M):                               # counts 1, 2, ... in turn, the last block among the kept ones
            mask[h, u, rng.permutation(s.M)[:1 + (u + h) % s.M]] = 1
            mask[h, u, s.M - 1] = 1
    mask[0, 0] = 1                                         # dense
    if s.M > 2:
        mask[1, 1] = 0                                     # empty
    o, lse = G.gpu_attn(g, P.DFS_F32, *(torch.from_numpy(x).cuda() for x in (q, k, v)), G.upload_mask(mask))
    o, lse = o.cpu().numpy(), lse.cpu().numpy()
    for h in range(2):
        for u in range(s.M):
            rows = slice(u * B, u * B + valid[u])
            if not mask[h, u].any():
                assert not o[h, rows].any() and np.isneginf(lse[h, rows]).all()
                continue
            want, want_lse = O.sparse_attn_block(*(x[h] for x in clean), np.nonzero(mask[h, u])[0], valid, B, u, 1.0 / np.sqrt(d))
            assert np.abs(o[h, rows] - want[:valid[u]]).max() <= 1e-4
            assert np.abs(lse[h, rows] - want_lse[:valid[u]]).max() <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale", [0.0, -0.125, 0.125])
def test_f32_forward_takes_any_scale(d, scale):
    """dfs_forward takes scales that are not positive; ragged and text blocks, whose pads are masked, among the kept."""
    g = P.Geom(1, 3, 67, 40, 2, d, 64, 16)
    s = P.dfs_geom_sizes(g)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    q, k, v = (torch.randn(2, s.N, d, generator=gen, device="cuda") for _ in range(3))
    perm_pad, inv, _ = G.gpu_perm(g)
    st = G.upload_mask(np.ones((2, s.M, s.M), dtype=np.uint8))
    o = torch.full_like(q, float("nan"))
    P.dfs_forward(g, P.DFS_F32, q, k, v, perm_pad, inv, False, P.DFS_SELECT_TOPK, 0.5, 0.0, st, scale, o,
                  G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD)))
    want = torch.softmax(q.double() @ k.double().transpose(1, 2) * scale, -1) @ v.double()
    assert (o - want).abs().max() <= 1e-4
