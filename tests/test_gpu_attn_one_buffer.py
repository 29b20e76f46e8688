"""bf16 attention at d = 128 with blocks of 64: above 512 work-groups the kernel keeps one tile buffer each for K and V, whose
halves take turns.  The arithmetic and its order are those of the form with two buffers, so the same two heads give the same
bits repeated over 257 to 512 work-groups (two buffers) and over more (one): lists of every length from none to all blocks, a
ragged last video block, text, with and without log-sum-exp, in the reordered and the source layout."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("n_video,n_text", [(64, 0), (40, 0), (5 * 64 - 23, 0), (12 * 64, 70), (20 * 64 - 4, 64)])
def test_same_bits_as_with_two_buffers(n_video, n_text):
    W = next(w for w in range(512, 0, -1) if n_video % w == 0 and n_video // w <= 512)
    geom = lambda copies: P.Geom(1, n_video // W, W, n_text, 2 * copies, 128, 64, 16)  # noqa: E731
    s = P.dfs_geom_sizes(geom(1))
    fewer, more = 512 // (2 * s.M), 512 // (2 * s.M) + 1
    few, many = geom(fewer), geom(more)
    assert 256 < 2 * fewer * s.M <= 512 < 2 * more * s.M
    rng = np.random.default_rng(n_video)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_video)
    q, k, v = (torch.randn(2, s.N_pad, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    k[:, ::7] *= 4                                         # rows outgrow their reference now and then
    mask = np.zeros((2, s.M, s.M), dtype=np.uint8)
    for h in range(2):
        for u in range(s.M):
            mask[h, u, rng.permutation(s.M)[:(u + h) % (s.M + 1)]] = 1
    st = G.upload_mask(mask, K_max=s.M)
    st.kv_cnt[:, 0] = s.M                                  # one dense row
    rep = lambda x, copies: x.repeat(copies, *([1] * (x.dim() - 1))).contiguous()  # noqa: E731
    real = torch.zeros(s.N_pad, dtype=torch.bool, device="cuda")
    real[:n_video] = True
    real[s.M_v * 64:s.M_v * 64 + n_text] = True
    perm_pad, inv, _ = G.gpu_perm(geom(1))
    src = torch.empty(2, s.N, 128, dtype=torch.bfloat16, device="cuda")
    P.dfs_unperm(geom(1), P.DFS_BF16, q, inv, src)
    got = []
    for g, copies in ((few, fewer), (many, more)):
        x = [rep(t, copies) for t in (q, k, v, src)]
        m = P.MaskState(rep(st.kv_idx, copies), rep(st.kv_cnt, copies), None, None, s.M)
        plain, _ = G.gpu_attn(g, P.DFS_BF16, *x[:3], m, want_lse=False)
        with_lse, lse = G.gpu_attn(g, P.DFS_BF16, *x[:3], m, want_lse=True)
        gathered = torch.empty_like(x[3])
        P.dfs_sparse_attn_fwd_src(g, P.DFS_BF16, x[3], perm_pad, x[1], x[2], m.kv_idx, m.kv_cnt, s.M, 128 ** -0.5, gathered)
        got.append((plain[:, real], with_lse[:, real], lse[:, real], gathered))
    for a, b in zip(*got):
        assert torch.isfinite(a[:2].float()).all() or a.dtype == torch.float32     # log-sum-exps of empty rows are -inf
        for c in range(more):
            assert torch.equal(b[2 * c:2 * c + 2], a[:2])
