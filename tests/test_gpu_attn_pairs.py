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


def _left_over(s, heads):
    """The rule for blocks that the pairs' full rounds leave: {(head, video block)}, how many an XCD (counting places that a shorter eighth does not
    fill) and how many work-groups to each."""
    eighth, text = ((s.M_v + 1) // 2 + 7) // 8, -(-heads * -(-s.M_x // 2) // 8)
    first, slots = (text + heads * eighth) // 32 * 32 - text, heads * eighth
    left = {(i // eighth, 2 * (x * eighth + i % eighth) + e) for x in range(8) for i in range(first, slots) for e in (0, 1)}
    rows = 2 * (slots - first)
    return {(h, u) for h, u in left if u < s.M_v}, rows, min(64 // rows, 4) if 0 < rows <= 32 else 1


def _differing(out, want, perm_pad, g, s):
    """{(head, block)} with a row that is not the same bits."""
    rows = G.gpu_permute(g, P.DFS_BF16, (out.view(torch.int16) != want.view(torch.int16)).to(torch.bfloat16), perm_pad)
    return {tuple(x) for x in rows.view(g.heads, s.M, -1).any(-1).nonzero().tolist()}


@pytest.mark.parametrize("T,H,W,n_text,heads,rows,text_splits", [
    (4, 132, 128, 0, 5, 10, 1),        # 528 blocks, 33 pairs an XCD and head: five pairs an XCD are left
    (4, 128, 130, 0, 5, 10, 1),        # 520, seven XCDs with as many and one with less
    (4, 129, 130, 0, 7, 14, 1),        # 525, the last one alone
    (4, 129, 130, 0, 14, 28, 1),       # two work-groups each
    (2, 127, 258, 300, 5, 4, 58),      # 512 + 3 text blocks: text rows in pairs, and split where a head's first rows are not dense
])
def test_blocks_left_over_are_shared(T, H, W, n_text, heads, rows, text_splits):
    """dfs_forward: the blocks of dense pairs that are left over, all of them and no other video block, are shared by several work-groups each, whoever
    merges; all other rows are the staged calls' bit for bit.  Shared rows differ by rounding: two results rounded to bf16 on their own, the suite's
    bound, over those rows alone."""
    g = P.Geom(T, H, W, n_text, heads, 128, 128, 32)
    s = P.dfs_geom_sizes(g)
    left, per_xcd, splits = _left_over(s, heads)
    assert per_xcd == rows and splits > 1 and heads * s.M >= 2048
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    perm_pad, inv, _ = G.gpu_perm(g)
    src = [torch.randn(heads, s.N, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3)]
    q, k, v = (G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in src)
    K_max = 9
    idx = torch.randint(0, s.M, (heads, s.M, K_max), generator=gen, device="cuda", dtype=torch.int32)
    cnt = torch.full((heads, s.M), s.M, dtype=torch.int32, device="cuda")
    cnt[heads - 1, :s.M_v:11] = 2                          # a head whose text rows are not in pairs
    dense = {tuple(x) for x in (cnt[:, :s.M_v] == s.M).nonzero().tolist()}
    want = torch.empty_like(q)
    P.dfs_sparse_attn_fwd(g, P.DFS_BF16, q, k, v, idx, cnt, K_max, 128 ** -0.5, want)
    want = G.gpu_unperm(g, P.DFS_BF16, want, inv)
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16))
    probe = torch.zeros(3, dtype=torch.int64, device="cuda")
    outs = []
    for fill in (255, 127):
        ws.fill_(fill)
        out = torch.full_like(src[0], float("nan"))
        step = lambda: P.dfs_forward(g, P.DFS_BF16, *src, perm_pad, inv, False, P.DFS_SELECT_TOPK, 0.0, 0.0,  # noqa: E731
                                     P.MaskState(idx, cnt, None, None, K_max), 128 ** -0.5, out, ws)
        assert G.kernels_of(step) == ["clear_tickets_kernel", "attn_pairs_kernel<128, 0, 1>", "attn_rest_kernel<128, 128, 0, 1, 1>"]
        P.dfs_attn_clock_probe(probe.zero_())
        try:
            step()
            torch.cuda.synchronize()
        finally:
            P.dfs_attn_clock_probe(None)
        outs.append(out)
    assert torch.equal(*outs)                              # whoever merges
    pair = lambda b: {(b[0], u) for u in (b[1] & ~1, b[1] | 1) if u < s.M_v}  # noqa: E731
    paired = {b for b in dense if pair(b) <= dense}
    shared = left & paired
    text = {(heads - 1, u) for u in range(s.M_v, s.M)}     # split, not in pairs
    other = _differing(outs[0], want, perm_pad, g, s)
    assert other == shared | text, (sorted(shared | text - other), sorted(other - shared - text))
    # work-groups: one to a pair in the full rounds and to a block that is in no pair, as many as share it to the others
    in_rounds = {(h, u & ~1) for h, u in paired - left}
    assert int(probe[2]) == len(in_rounds) + heads * s.M_v - len(paired) + len(shared) * splits + (heads - 1) * -(-s.M_x // 2) + s.M_x * text_splits
    merged = torch.zeros(heads, s.M, 128, dtype=torch.bool, device="cuda")
    for h, u in shared | text:
        merged[h, u] = True
    merged = G.gpu_unperm(g, P.DFS_BF16, merged.view(heads, s.N_pad, 1).expand(-1, -1, 128).to(torch.bfloat16).contiguous(), inv)[:, :, 0] > 0
    a, b = outs[0][merged].double(), want[merged].double()
    assert float((a - b).norm() / b.norm()) <= 7.5e-3 and float(((a - b).norm(dim=-1) / b.norm(dim=-1)).max()) <= 2 * 7.5e-3
    if not n_text:                                         # a refresh step that keeps every block: the same sharing, its tickets cleared by the pooling
        idx2, cnt2 = torch.full((heads, s.M, s.M), -1, dtype=torch.int32, device="cuda"), torch.full_like(cnt, -1)
        full = []
        for refresh in (True, False):
            ws.fill_(255)
            out = torch.full_like(src[0], float("nan"))
            step = lambda: P.dfs_forward(g, P.DFS_BF16, *src, perm_pad, inv, refresh, P.DFS_SELECT_TOPK, 0.0, 0.0,  # noqa: E731
                                         P.MaskState(idx2, cnt2, None, None, s.M), 128 ** -0.5, out, ws)
            assert G.kernels_of(step)[-2:] == ["attn_pairs_kernel<128, 0, 1>", "attn_rest_kernel<128, 128, 0, 1, 1>"]
            step()
            full.append(out)
        assert bool((cnt2 == s.M).all()) and torch.equal(*full)
        assert left <= _differing(full[0], want, perm_pad, g, s)


@pytest.mark.parametrize("heads", [5, 9])                  # five rounds of work-groups and a part, whose rows are shared; nine and a part, which are not
def test_reuse_of_masked_lists_gives_the_refresh(heads):
    """Lists that drop blocks: a reuse step, which looks for dense pairs, and the refresh step that made them, which does not, share the same rows."""
    g = P.Geom(4, 128, 130, 0, heads, 128, 128, 32)
    s = P.dfs_geom_sizes(g)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    perm_pad, inv, _ = G.gpu_perm(g)
    src = [torch.randn(g.heads, s.N, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3)]
    K_max = P.dfs_keep_count(0.9, s.M_v)
    i32 = dict(dtype=torch.int32, device="cuda")
    st = P.MaskState(torch.zeros((g.heads, s.M, K_max), **i32), torch.zeros((g.heads, s.M), **i32), None, None, K_max)
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16))
    outs = []
    for refresh in (True, False):
        out = torch.full_like(src[0], float("nan"))
        step = lambda: P.dfs_forward(g, P.DFS_BF16, *src, perm_pad, inv, refresh, P.DFS_SELECT_TOPK, 0.9, 0.0, st, 128 ** -0.5, out, ws)  # noqa: E731
        assert any("pairs" in n for n in G.kernels_of(step)) == (not refresh)
        step()
        outs.append(out)
    assert torch.equal(*outs)
