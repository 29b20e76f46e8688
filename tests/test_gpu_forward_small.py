"""A refresh step of a small fp32 problem is one kernel (forward_small_kernel): lists, counts, masks and output bit for bit those of the staged
calls.  The limits of its range and the first shapes beyond them, every number of sub-blocks, ragged blocks, text, a row's own count; the calls that
keep their three kernels; orders with entries that are none; a reuse step that gathers its keys and values."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


def _step(g, qkv, perm_pad, inv, refresh, mode, sparsity, mass, st, out, run=True):
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD))
    call = lambda: P.dfs_forward(g, P.DFS_F32, *qkv, perm_pad, inv, refresh, mode, sparsity, mass, st, g.d ** -0.5, out, ws)  # noqa: E731
    names = G.kernels_of(call)
    if run:
        call()
    return names


def _state(g, s, K_max, fill=-1):
    i32 = dict(dtype=torch.int32, device="cuda")
    return P.MaskState(torch.full((g.heads, s.M, K_max), fill, **i32), torch.full((g.heads, s.M), fill, **i32),
                       torch.full((g.heads, s.M, s.M), 9, dtype=torch.uint8, device="cuda"), torch.full((g.heads,), fill, **i32), K_max)


@pytest.mark.parametrize("T,H,W,n_text,heads,d,B,r,small", [
    (1, 1, 3, 0, 1, 64, 64, 4, True), (4, 8, 8, 0, 2, 64, 64, 4, True), (1, 19, 27, 5, 3, 128, 64, 1, False), (1, 19, 26, 5, 3, 128, 64, 2, True),
    (2, 16, 32, 0, 4, 64, 128, 8, True),                   # 1 024 tokens, 64 sub-blocks, 128 work-groups: the video's limits
    (1, 25, 41, 0, 1, 64, 64, 4, False),                   # 1 025
    (1, 25, 40, 0, 1, 64, 64, 8, False),                   # 128 sub-blocks
    (1, 23, 29, 1344, 1, 64, 64, 1, True),                 # 2 048 rows, most of them text
    (1, 23, 29, 1345, 1, 64, 64, 1, False),
    (1, 21, 24, 0, 16, 128, 128, 8, True), (1, 21, 24, 0, 17, 128, 128, 8, False),                 # 256 work-groups and more
    (3, 7, 11, 70, 5, 128, 64, 8, True), (1, 9, 70, 129, 2, 64, 128, 2, True),
    (1, 16, 30, 40, 2, 128, 128, 2, True), (1, 16, 30, 40, 2, 64, 128, 1, True), (1, 16, 30, 40, 2, 128, 128, 1, False)])      # the longest sub-blocks
def test_same_as_staged(T, H, W, n_text, heads, d, B, r, small):
    g = P.Geom(T, H, W, n_text, heads, d, B, B // r)
    s = P.dfs_geom_sizes(g)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * W + r)
    qkv = [torch.randn(heads, s.N, d, generator=gen, device="cuda") for _ in range(3)]
    perm_pad, inv, _ = G.gpu_perm(g)
    damaged = perm_pad.clone()
    bad = torch.tensor([-1, -5, s.N, 2 ** 31 - 1, -2 ** 31], device="cuda", dtype=torch.int32)
    damaged[::13] = bad[torch.arange(damaged[::13].numel(), device="cuda") % 5]
    for order in (perm_pad, damaged):
        rows = order[(order >= 0) & (order < s.N)].long()
        qp, kp, vp = (G.gpu_permute(g, P.DFS_F32, x, order) for x in qkv)
        score = G.gpu_score(g, P.DFS_F32, qp, kp)
        for mode, sparsity, mass in ((P.DFS_SELECT_TOPK, 0.6, 0.0), (P.DFS_SELECT_MASS_ROW, 0.95, 0.8), (P.DFS_SELECT_TOPK, 0.0, 0.0)):
            K_max = s.M if mode != P.DFS_SELECT_TOPK else P.dfs_keep_count(sparsity, s.M_v) + s.M_x
            want = G.gpu_select(g, score, mode, sparsity, mass, K_max=K_max)
            want_o = G.gpu_attn(g, P.DFS_F32, qp, kp, vp, want)[0]
            real = ((order >= 0) & (order < s.N)).nonzero()[:, 0]
            st, out = _state(g, s, K_max), torch.full_like(qkv[0], float("nan"))
            names = _step(g, qkv, order, inv, True, mode, sparsity, mass, st, out)
            assert (names == [f"forward_small_kernel<{d}, {r}>"]) == small, names
            for name in ("kv_cnt", "mask", "k_head"):
                assert torch.equal(getattr(st, name), getattr(want, name)), (name, mode)
            listed = torch.arange(K_max, device="cuda") < st.kv_cnt[:, :s.M_v, None]       # text rows carry no list
            assert torch.equal(torch.where(listed, st.kv_idx[:, :s.M_v], -1), torch.where(listed, want.kv_idx[:, :s.M_v], -1))
            assert torch.equal(out[:, rows], want_o[:, real])
            again = torch.full_like(out, float("nan"))                                     # reuse step
            names = _step(g, qkv, order, inv, False, mode, sparsity, mass, st, again)
            assert (names == [f"attn_f32_kernel<{d}, 1>"]) == (4 * heads * d * s.N_pad ** 2 <= 2 ** 31), names
            assert torch.equal(again[:, rows], want_o[:, real])


@pytest.mark.parametrize("over", [0, 1, 2])
@pytest.mark.parametrize("r", [1, 4])
def test_output_over_an_input(over, r):
    g = P.Geom(1, 16, 24, 20, 2, 64, 64, 64 // r)
    s = P.dfs_geom_sizes(g)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(over)
    qkv = [torch.randn(2, s.N, 64, generator=gen, device="cuda") for _ in range(3)]
    perm_pad, inv, _ = G.gpu_perm(g)
    K_max = P.dfs_keep_count(0.5, s.M_v) + s.M_x
    want = torch.empty_like(qkv[0])
    st = _state(g, s, K_max)
    assert _step(g, qkv, perm_pad, inv, True, P.DFS_SELECT_TOPK, 0.5, 0.0, st, want) == [f"forward_small_kernel<64, {r}>"]
    for refresh in (True, False):
        x = [t.clone() for t in qkv]
        names = _step(g, x, perm_pad, inv, refresh, P.DFS_SELECT_TOPK, 0.5, 0.0, st, x[over])
        assert not any("small" in n and "forward" in n for n in names)
        assert torch.equal(x[over], want)
    head = _state(g, s, s.M)
    assert len(_step(g, qkv, perm_pad, inv, True, P.DFS_SELECT_MASS_HEAD, 0.9, 0.9, head, want, run=False)) > 1
