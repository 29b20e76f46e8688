"""dfs_forward shares the query blocks of the last round of work-groups between several (bf16, above 512 query blocks).  Against the
staged kernel, which keeps every block whole, on the same lists: shapes just above one and two rounds for each d and B, in each
order of work-groups (heads in turn, all XCDs on one head, text in front), lists of equal and unequal length, shorter than the
pieces and empty.  Each side is within 1.9e-3 (2-norm, relative) of the exact result through the rounding of weights and result,
so they differ by less than 4e-3; repeated calls give the same bits.  Every shape is checked to share its last round by the
library's rule, and the one with whole text blocks to have one of them there."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


def _shared_tail(g, s, K_max, text_splits):
    """The rule of tail_split for these shapes: (work-groups to a query block of the last round, text blocks there)."""
    M_x, chunk, total = s.M_x, -(-s.M_v // 8), g.heads * s.M
    mapping = 2 if chunk >= 64 else 3 if text_splits > 1 else 1
    one_buffer = g.d == 128 and g.B == 64 and total + g.heads * M_x * (text_splits - 1) > 512 and mapping != 2
    text_slots = -(-g.heads * M_x * text_splits // 8) if mapping > 1 else 0
    per_xcd = g.heads * chunk if mapping == 2 else -(-g.heads * s.M_v // 8) if mapping == 3 else -(-total // 8)
    slots = 32 * ((3 if g.d == 64 else 2) if g.B == 128 else 4 if g.d == 64 or one_buffer else 2)
    order = text_slots + per_xcd
    full = order // slots * slots
    rows = order - full
    if full == 0 or rows == 0 or full < text_slots or full > (2 if one_buffer else 8) * slots:
        return 1, 0
    pieces = (K_max if K_max < s.M else s.M // 3) // (4 if full == slots else 6)
    splits = min(slots // rows, 4, pieces)
    last = [x * per_xcd + slot for x in range(8) for slot in range(full, order) if x * per_xcd + slot < total]
    text = sum(i % s.M < M_x for i in last) if mapping == 1 else 0
    return (splits, text) if splits >= (3 if g.d == 128 and g.B == 128 else 2) else (1, 0)


@pytest.mark.parametrize("d,B,T,H,W,n_text,heads,keep", [
    (128, 128, 5, 16, 64, 0, 13, 20),       # 520 query blocks of 40: one round and a bit
    (128, 128, 9, 31, 33, 0, 15, 30),       # 1080, the last one ragged
    (128, 128, 2, 260, 127, 0, 1, 60),      # 516 of one head: all XCDs on it
    (128, 128, 5, 37, 43, 100, 9, 30),      # text, split, in front
    (64, 128, 5, 32, 64, 0, 10, 20),        # 800
    (64, 128, 5, 32, 64, 40, 30, 40),       # 2 430 with one text block each, whole, one of them in the last round
    (64, 128, 1, 27, 41, 9, 81, 9),         # 810, likewise: blocks of a sequence too short to split its text
    (64, 64, 5, 16, 64, 0, 13, 24),         # 1 040
    (128, 64, 4, 31, 65, 0, 9, 32),         # 1 134, one buffer
])
def test_shared_tail_against_whole_blocks(d, B, T, H, W, n_text, heads, keep):
    g = P.Geom(T, H, W, n_text, heads, d, B, B // 4)
    s = P.dfs_geom_sizes(g)
    K_max = min(s.M, keep)
    splits, text = _shared_tail(g, s, K_max, 3 if n_text == 100 else 1)
    print(f"d={d} B={B} {T}x{H}x{W}+{n_text} x {heads}: {splits} work-groups to a block, {text} text blocks", flush=True)
    assert heads * s.M >= 512 and splits > 1 and (text > 0) == (n_text in (40, 9))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(heads * d + B)
    q, k, v = (torch.randn(heads, s.N, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    k[:, ::5] *= 3
    perm_pad, inv, _ = G.gpu_perm(g)
    idx = torch.rand(heads, s.M, s.M, generator=gen, device="cuda").argsort(-1)[:, :, :K_max].sort(-1)[0].int().contiguous()
    cnt = torch.full((heads, s.M), K_max, dtype=torch.int32, device="cuda")
    kp, vp = (G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in (k, v))
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16))
    for lists in ("equal", "unequal", "dense"):
        if lists == "unequal":
            cnt.copy_(torch.randint(0, K_max + 1, cnt.shape, generator=gen, device="cuda"))
            cnt[:, -3:] = torch.tensor([0, 1, min(2, K_max)])           # the blocks dealt last or first, either way
            cnt[:, :3] = torch.tensor([2, 0, 1])
        elif lists == "dense":
            cnt.fill_(s.M)
        if n_text:
            cnt[:, s.M_v:] = s.M
        want = torch.empty_like(q)
        P.dfs_sparse_attn_fwd_src(g, P.DFS_BF16, q, perm_pad, kp, vp, idx, cnt, K_max, d ** -0.5, want)
        out = []
        for _ in range(2):
            ws.fill_(0x7F)                                             # tickets and partial rows of an earlier call are no help
            o = torch.full_like(q, 7.0)
            P.dfs_forward(g, P.DFS_BF16, q, k, v, perm_pad, inv, False, P.DFS_SELECT_TOPK, 0.5, 0.0, P.MaskState(idx, cnt, None, None, K_max),
                          d ** -0.5, o, ws)
            out.append(o)
        assert torch.equal(*out)
        a, b = out[0].double(), want.double()
        rows = b.norm(dim=-1)
        assert float((a - b).norm() / b.norm()) < 4e-3
        assert float(((a - b).norm(dim=-1) / rows.clamp_min(1e-30))[rows > 0].max()) < 3e-2      # no row is off by more than a few roundings
        assert bool((a[rows == 0] == 0).all())                          # empty lists give zero rows
