"""dfs_forward's bf16 attention gathers keys and values from the tensors in source order.  Against the staged calls, which reorder
them first, bit for bit, for every instance of the kernel that does so and whose rows are not shared between work-groups: lists of
every length from none to all blocks, ragged last blocks, text, orders of every kind and orders with entries that are none."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402

# T, H, W, n_text, heads, d, B: work-groups and list room that make each instance
SHAPES = [
    (1, 1, 5, 0, 1, 64, 64),          # a lone ragged block, two wave groups
    (2, 5, 75, 3, 2, 64, 64),         # two wave groups, text
    (1, 16, 85, 0, 25, 64, 64),       # 550 work-groups: one group, the last round whole
    (2, 5, 77, 40, 2, 64, 128),       # two wave groups of four
    (1, 31, 57, 0, 19, 64, 128),      # 266 work-groups: one group
    (2, 5, 75, 3, 2, 128, 64),        # two wave groups, two buffers
    (3, 7, 61, 0, 15, 128, 64),       # 315 work-groups: one group, two buffers
    (1, 32, 64, 0, 57, 128, 64),      # 1 824 work-groups: one buffer
    (1, 17, 47, 9, 112, 128, 64),     # the same with a ragged block and text (fewer than 16 blocks: whole rows): 1 568
    (1, 1, 9, 0, 600, 128, 64),       # one buffer, a lone ragged block
    (2, 5, 77, 40, 2, 128, 128),      # one group, lists of up to 16
    (2, 41, 49, 0, 3, 128, 128),      # two wave groups, lists of 17 and more
]


def _problem(T, H, W, n_text, heads, d, B, seed=5):
    g = P.Geom(T, H, W, n_text, heads, d, B, B // 4)
    s = P.dfs_geom_sizes(g)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    q, k, v = (torch.randn(heads, s.N, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    k[:, ::7] *= 4                                         # rows outgrow their reference now and then
    rng = np.random.default_rng(seed)
    mask = np.zeros((heads, s.M, s.M), dtype=np.uint8)
    for h in range(heads):
        for u in range(s.M):
            mask[h, u, rng.permutation(s.M)[:(u + h) % (s.M + 1)]] = 1
    st = G.upload_mask(mask, K_max=s.M)
    perm_pad, inv, _ = G.gpu_perm(g)
    return g, s, (q, k, v), st, perm_pad, inv


def _staged(g, s, qkv, st, perm_pad, out):
    """The kept lists' attention with K and V reordered by calls of their own, from the same positions."""
    kp, vp = (G.gpu_permute(g, P.DFS_BF16, x, perm_pad) for x in qkv[1:])
    P.dfs_sparse_attn_fwd_src(g, P.DFS_BF16, qkv[0], perm_pad, kp, vp, st.kv_idx, st.kv_cnt, st.K_max, g.d ** -0.5, out)
    return out


def _forward(g, qkv, st, perm_pad, inv, out, ws=None):
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16)) if ws is None else ws
    P.dfs_forward(g, P.DFS_BF16, *qkv, perm_pad, inv, False, P.DFS_SELECT_TOPK, 0.5, 0.0, st, g.d ** -0.5, out, ws)
    return out


def _same(a, b):
    return torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("shape", SHAPES)
def test_same_bits_as_reordered(shape):
    g, s, qkv, st, perm_pad, inv = _problem(*shape)
    empty = torch.full_like(qkv[0], float("nan"))
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


@pytest.mark.parametrize("shape", [SHAPES[i] for i in (1, 4, 6, 8, 10)])
def test_positions_that_are_none_read_as_zeros(shape):
    g, s, qkv, st, perm_pad, inv = _problem(*shape)
    order = perm_pad.clone()
    bad = torch.tensor([-1, -2, -(2 ** 31), s.N, s.N + 1, 2 ** 24, 2 ** 24 + 1, 2 ** 25 + 3, 2 ** 31 - 1], device="cuda")
    at = torch.arange(3, s.N_pad, 29, device="cuda")
    order[at] = bad[torch.arange(at.numel(), device="cuda") % bad.numel()].to(torch.int32)
    zero = torch.zeros_like(qkv[0])
    assert _same(_forward(g, qkv, st, order, inv, zero.clone()), _staged(g, s, qkv, st, order, zero.clone()))


@pytest.mark.parametrize("over", ["k", "v", "k_end", "v_start"])
@pytest.mark.parametrize("shape", [SHAPES[4], SHAPES[8]])
def test_output_over_the_keys_or_values(shape, over):
    g, s, qkv, st, perm_pad, inv = _problem(*shape)
    want = _forward(g, qkv, st, perm_pad, inv, torch.empty_like(qkv[0]))
    n = qkv[0].numel()
    room = torch.empty(3 * n, dtype=torch.bfloat16, device="cuda")
    at = room[n:2 * n].view_as(qkv[0])
    at.copy_(qkv[1] if over[0] == "k" else qkv[2])
    first = {"k": n, "v": n, "k_end": 2 * n - 64, "v_start": 64}[over]
    out = room[first:first + n].view_as(qkv[0])
    inputs = (qkv[0], at, qkv[2]) if over[0] == "k" else (qkv[0], qkv[1], at)
    assert _same(_forward(g, inputs, st, perm_pad, inv, out), want)
