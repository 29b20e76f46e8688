"""dfs_forward's bf16 attention gathers keys and values from the tensors in source order.  Bit for bit, for every instance of the
kernel that a geometry takes there, against a call that reorders them first: the staged ones where every row has one work-group, dfs_forward with the
output over its keys where rows are shared.  Lists of every length from none to all blocks, ragged last blocks, text, orders of
every kind and orders with entries that are none.  Every shape is checked to launch the instance that it stands for."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402

# T, H, W, n_text, heads, d, B: work-groups and list room that make each instance; its wave groups, whether it has one tile buffer
SHAPES = [
    ((1, 1, 5, 0, 1, 64, 64), 2, 0),          # a lone ragged block, two wave groups
    ((2, 5, 75, 3, 2, 64, 64), 2, 0),         # two wave groups, text
    ((1, 16, 85, 0, 25, 64, 64), 1, 0),       # 550 work-groups: one group, the last round whole
    ((2, 5, 77, 40, 2, 64, 128), 2, 0),       # two wave groups of four
    ((1, 31, 57, 0, 19, 64, 128), 1, 0),      # 266 work-groups: one group
    ((2, 5, 75, 3, 2, 128, 64), 2, 0),        # two wave groups, two buffers
    ((3, 7, 61, 0, 15, 128, 64), 1, 0),       # 315 work-groups: one group, two buffers
    ((1, 32, 64, 0, 57, 128, 64), 1, 1),      # 1 824 work-groups: one buffer
    ((1, 17, 47, 9, 112, 128, 64), 1, 1),     # the same with a ragged block and text (fewer than 16 blocks: whole rows): 1 568
    ((1, 1, 9, 0, 600, 128, 64), 1, 1),       # one buffer, a lone ragged block
    ((2, 5, 77, 40, 2, 128, 128), 1, 0),      # one group, lists of up to 16
    ((2, 41, 49, 0, 3, 128, 128), 2, 0),      # two wave groups, lists of 17 and more
    ((1, 41, 61, 0, 15, 128, 128), 1, 0),     # 300 work-groups: one group, lists of up to 20
    ((2, 127, 255, 0, 1, 128, 128), 1, 0),    # 507 blocks: all XCDs on one head, lists of up to 507, the last block ragged
]


def _problem(T, H, W, n_text, heads, d, B, K_max=None, seed=5):
    g = P.Geom(T, H, W, n_text, heads, d, B, B // 4)
    s = P.dfs_geom_sizes(g)
    K_max = s.M if K_max is None else K_max
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    q, k, v = (torch.randn(heads, s.N, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    k[:, ::7] *= 4                                         # rows outgrow their reference now and then
    rng = np.random.default_rng(seed)
    mask = np.zeros((heads, s.M, s.M), dtype=np.uint8)
    for h in range(heads):
        for u in range(s.M):
            mask[h, u, rng.permutation(s.M)[:(u + h) % (K_max + 1)]] = 1
    mask[:, s.M_v:] = 1 if K_max < s.M else mask[:, s.M_v:]     # text rows as the library keeps them
    st = G.upload_mask(mask, K_max=K_max)
    perm_pad, inv, _ = G.gpu_perm(g)
    return g, s, (q, k, v), st, perm_pad, inv


def _staged(g, s, qkv, st, perm_pad, out):
    """The kept lists' attention with K and V reordered by calls of their own, from the same positions."""
    kp, vp = (G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in qkv[1:])
    P.dfs_sparse_attn_fwd_src(g, P.DFS_BF16, qkv[0], perm_pad, kp, vp, st.kv_idx, st.kv_cnt, st.K_max, g.d ** -0.5, out)
    return out


def _forward(g, qkv, st, perm_pad, inv, out, refresh=False):
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16))
    ws.fill_(255)
    P.dfs_forward(g, P.DFS_BF16, *qkv, perm_pad, inv, refresh, P.DFS_SELECT_TOPK, 0.5, 0.0, st, g.d ** -0.5, out, ws)
    return out


def _over_the_keys(g, qkv, st, perm_pad, inv, refresh=False):
    """dfs_forward with the output over its keys, which it then reorders, and the values, before the first row is written."""
    k = qkv[1].clone()
    return _forward(g, (qkv[0], k, qkv[2]), st, perm_pad, inv, k, refresh)


def _attn(g, groups, one_buffer, shared, gathers):
    return f"attn_bf16_kernel<{g.d}, {g.B}, 0, {groups}, {one_buffer}, {shared}, {gathers}>"


def _same(a, b):
    return torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("shape,groups,one_buffer", SHAPES)
def test_same_bits_as_reordered(shape, groups, one_buffer):
    g, s, qkv, st, perm_pad, inv = _problem(*shape)
    empty = torch.full_like(qkv[0], float("nan"))
    assert G.kernels_of(lambda: _forward(g, qkv, st, perm_pad, inv, empty.clone()))[-1] == _attn(g, groups, one_buffer, 0, 1)
    # the call before leaves NaN wherever a tile may have been
    nan = torch.full_like(qkv[0], float("nan"))
    _forward(g, (nan, nan, nan), st, perm_pad, inv, empty.clone())
    want = _staged(g, s, qkv, st, perm_pad, empty.clone())
    _forward(g, (nan, nan, nan), st, perm_pad, inv, empty.clone())
    got = _forward(g, qkv, st, perm_pad, inv, empty.clone())
    assert torch.isfinite(got.float()).all()
    assert _same(got, want)
    # any other order of the real tokens, pads where they are
    real = perm_pad >= 0
    for order in range(2):
        other = perm_pad.clone()
        if order == 0:
            other[real] = torch.arange(s.N, dtype=torch.int32, device="cuda")
        else:
            gen = torch.Generator(device="cuda")
            gen.manual_seed(3)
            other[real] = torch.randperm(s.N, generator=gen, device="cuda").to(torch.int32)
        assert _same(_forward(g, qkv, st, other, inv, empty.clone()), _staged(g, s, qkv, st, other, empty.clone()))


def _with_positions_that_are_none(s, perm_pad):
    order = perm_pad.clone()
    bad = torch.tensor([-1, -2, -(2 ** 31), s.N, s.N + 1, 2 ** 24, 2 ** 24 + 1, 2 ** 25 + 3, 2 ** 31 - 1], device="cuda")
    at = torch.arange(3, s.N_pad, 29, device="cuda")
    order[at] = bad[torch.arange(at.numel(), device="cuda") % bad.numel()].to(torch.int32)
    return order


@pytest.mark.parametrize("shape", [SHAPES[i][0] for i in (1, 4, 6, 8, 10, 13)])
def test_positions_that_are_none_read_as_zeros(shape):
    g, s, qkv, st, perm_pad, inv = _problem(*shape)
    order = _with_positions_that_are_none(s, perm_pad)
    zero = torch.zeros_like(qkv[0])
    assert _same(_forward(g, qkv, st, order, inv, zero.clone()), _staged(g, s, qkv, st, order, zero.clone()))


# T, H, W, n_text, heads, d, B, K_max: shapes that share rows; wave groups, one tile buffer, whether the last round is shared (else
# only text rows are)
SHARED = [
    ((1, 32, 32, 1, 3, 64, 64, 6), 2, 0, 0),           # text over work-groups of two wave groups each
    ((1, 40, 51, 130, 2, 64, 128, 10), 2, 0, 0),
    ((1, 41, 27, 200, 1, 128, 64, 6), 2, 0, 0),
    ((1, 43, 48, 77, 24, 128, 128, 3), 1, 0, 0),
    ((1, 90, 80, 128, 2, 128, 128, 20), 2, 0, 0),
    ((5, 16, 64, 0, 13, 64, 64, 24), 1, 0, 1),         # the last round, 1 040 work-groups
    ((5, 32, 64, 40, 30, 64, 128, 40), 1, 0, 1),       # 2 430, a whole text block in the last round
    ((4, 31, 65, 0, 9, 128, 64, 32), 1, 1, 1),         # one buffer
    ((2, 260, 127, 0, 1, 128, 128, 60), 1, 0, 1),      # 516 of one head: all XCDs on it
    ((5, 37, 43, 100, 9, 128, 128, 30), 1, 0, 1),      # text and the last round
]


@pytest.mark.parametrize("shape,groups,one_buffer,tail", SHARED)
def test_shared_rows_same_bits_as_reordered(shape, groups, one_buffer, tail):
    g, s, qkv, st, perm_pad, inv = _problem(*shape)
    empty = torch.full_like(qkv[0], float("nan"))
    clear = "clear_tickets_kernel"                         # only where rows are shared
    assert G.kernels_of(lambda: _forward(g, qkv, st, perm_pad, inv, empty.clone()))[-2:] == [clear, _attn(g, groups, one_buffer, tail, 1)]
    assert G.kernels_of(lambda: _over_the_keys(g, qkv, st, perm_pad, inv))[-1] == _attn(g, groups, one_buffer, tail, 0)
    want = _over_the_keys(g, qkv, st, perm_pad, inv)
    assert torch.isfinite(want.float()).all()
    for _ in range(2):                                     # whoever merges
        assert _same(_forward(g, qkv, st, perm_pad, inv, empty.clone()), want)
    order = _with_positions_that_are_none(s, perm_pad)
    rows = order[(order >= 0) & (order < s.N)].long()      # the rows that are written
    assert _same(_forward(g, qkv, st, order, inv, empty.clone())[:, rows], _over_the_keys(g, qkv, st, order, inv)[:, rows])


@pytest.mark.parametrize("refresh", [False, True])
@pytest.mark.parametrize("over", ["k", "v", "k_end", "v_start"])
@pytest.mark.parametrize("shape", [SHAPES[4][0], SHAPES[8][0]])
def test_output_over_the_keys_or_values(shape, over, refresh):
    g, s, qkv, st, perm_pad, inv = _problem(*shape)
    want = _forward(g, qkv, st, perm_pad, inv, torch.empty_like(qkv[0]), refresh)
    n = qkv[0].numel()
    room = torch.empty(3 * n, dtype=torch.bfloat16, device="cuda")
    at = room[n:2 * n].view_as(qkv[0])
    at.copy_(qkv[1] if over[0] == "k" else qkv[2])
    first = {"k": n, "v": n, "k_end": 2 * n - 64, "v_start": 64}[over]
    out = room[first:first + n].view_as(qkv[0])
    inputs = (qkv[0], at, qkv[2]) if over[0] == "k" else (qkv[0], qkv[1], at)
    assert _same(_forward(g, inputs, st, perm_pad, inv, out, refresh), want)
