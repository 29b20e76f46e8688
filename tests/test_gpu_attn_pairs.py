"""Dense query blocks in pairs (attn_pairs_kernel), bit for bit against the blocks one by one: heads of one problem in one call, whose
dense rows are taken in pairs, against a call per head, too small for that.  An odd last block, text, the blocks behind the last full
round, and lists of which some are dense: both blocks of a pair, one of them, a head without dense video rows."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("T,H,W,n_text,heads,mixed", [
    (1, 181, 357, 0, 5, False),        # 505 blocks, the last ragged and alone in its pair: five full rounds
    (2, 127, 258, 300, 5, True),       # 512 + 3 text blocks, the last of each ragged; 2 round slots of an XCD left over
])
def test_same_bits_as_one_by_one(T, H, W, n_text, heads, mixed):
    g, one = (P.Geom(T, H, W, n_text, h, 128, 128, 32) for h in (heads, 1))
    s = P.dfs_geom_sizes(g)
    assert s.M_v > 504 and heads * s.M >= 2048
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H)
    perm_pad, inv, _ = G.gpu_perm(g)
    src = [torch.randn(heads, s.N, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3)]
    q, k, v = (G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in src)
    K_max = 9
    idx = torch.randint(0, s.M, (heads, s.M, K_max), generator=gen, device="cuda", dtype=torch.int32)
    cnt = torch.full((heads, s.M), s.M, dtype=torch.int32, device="cuda")
    if mixed:
        cnt[1, :s.M_v] = 5                                 # a head whose text rows alone are dense
        cnt[2, ::7] = 3                                    # one of a pair, both now and then
        cnt[3, 1::2] = 0
        cnt[4, s.M - 1] = 2
    call = lambda *a: P.dfs_sparse_attn_fwd(*a)  # noqa: E731
    scale = 128 ** -0.5
    for want_lse in (False, True):
        o, want = (torch.full_like(q, float("nan")) for _ in range(2))
        lse, want_l = (torch.full((heads, s.N_pad), float("nan"), device="cuda") if want_lse else None for _ in range(2))
        names = G.kernels_of(lambda: call(g, P.DFS_BF16, q, k, v, idx, cnt, K_max, scale, o, lse))
        assert names == [f"attn_pairs_kernel<128, {int(want_lse)}, 0>", f"attn_rest_kernel<128, 128, {int(want_lse)}, 0, 0>"]
        call(g, P.DFS_BF16, q, k, v, idx, cnt, K_max, scale, o, lse)
        for h in range(heads):
            assert not any("pairs" in n for n in G.kernels_of(lambda: call(one, P.DFS_BF16, q[h:h + 1], k[h:h + 1], v[h:h + 1], idx[h:h + 1], cnt[h:h + 1], K_max,
                                                                           scale, want[h:h + 1], want_l[h:h + 1] if want_lse else None)))
            call(one, P.DFS_BF16, q[h:h + 1], k[h:h + 1], v[h:h + 1], idx[h:h + 1], cnt[h:h + 1], K_max, scale, want[h:h + 1],
                 want_l[h:h + 1] if want_lse else None)
        assert torch.isfinite(want.float()).all()
        assert torch.equal(o.view(torch.int16), want.view(torch.int16))
        if want_lse:
            assert torch.equal(lse.view(torch.int32), want_l.view(torch.int32))
    if n_text:
        return                                             # dfs_forward shares rows there, which then round differently
    # source order: keys and values gathered
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16))
    st = P.MaskState(idx, cnt, None, None, K_max)
    out = torch.full_like(src[0], float("nan"))
    step = lambda: P.dfs_forward(g, P.DFS_BF16, *src, perm_pad, inv, False, P.DFS_SELECT_TOPK, 0.0, 0.0, st, scale, out, ws)  # noqa: E731
    assert G.kernels_of(step) == ["attn_pairs_kernel<128, 0, 1>", "attn_rest_kernel<128, 128, 0, 0, 1>"]
    step()
    assert torch.equal(out.view(torch.int16), G.gpu_unperm(g, P.DFS_BF16, want, inv).view(torch.int16))


def test_blocks_left_over_are_shared():
    """dfs_forward: 520 blocks of five heads leave five pairs an XCD over, which four work-groups share each; all other rows are the staged calls' bit
    for bit.  Shared rows differ by rounding: two results rounded to bf16 on their own, the suite's bound."""
    heads = 5
    g = P.Geom(4, 128, 130, 0, heads, 128, 128, 32)
    s = P.dfs_geom_sizes(g)
    assert s.M_v == 520
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    perm_pad, inv, _ = G.gpu_perm(g)
    src = [torch.randn(heads, s.N, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3)]
    q, k, v = (G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in src)
    idx = torch.randint(0, s.M, (heads, s.M, 9), generator=gen, device="cuda", dtype=torch.int32)
    cnt = torch.full((heads, s.M), s.M, dtype=torch.int32, device="cuda")
    cnt[4, ::11] = 9
    want = torch.empty_like(q)
    P.dfs_sparse_attn_fwd(g, P.DFS_BF16, q, k, v, idx, cnt, 9, 128 ** -0.5, want)
    want = G.gpu_unperm(g, P.DFS_BF16, want, inv)
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16))
    outs = []
    for _ in range(2):
        ws.fill_(255)
        out = torch.full_like(src[0], float("nan"))
        step = lambda: P.dfs_forward(g, P.DFS_BF16, *src, perm_pad, inv, False, P.DFS_SELECT_TOPK, 0.0, 0.0,  # noqa: E731
                                     P.MaskState(idx, cnt, None, None, 9), 128 ** -0.5, out, ws)
        assert G.kernels_of(step) == ["clear_tickets_kernel", "attn_pairs_kernel<128, 0, 1>", "attn_rest_kernel<128, 128, 0, 1, 1>"]
        step()
        outs.append(out)
    assert torch.equal(*outs)                              # whoever merges
    assert float((outs[0].double() - want.double()).norm() / want.double().norm()) <= 7.5e-3
    other = (outs[0] != want).any(2)                       # of 10 blocks an XCD, all of the last head
    assert int(other.sum()) <= 8 * 10 * 128 and not bool(other[:4].any())
