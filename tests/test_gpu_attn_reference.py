"""bf16 attention when a row's logits outgrow the reference its softmax started with: rows that grow slowly (the
reference moves along), in jumps, by far, only in the last block, and rows that fall.  Against the oracle under the same
lists, through the C ABI.  Then what following the reference is for: the rounding of the weights, rows without a finite
logit, large values."""
import math

import numpy as np
import pytest
import torch

from oracle import dfs_oracle as O
from workloads import to_bf16_bits
from workloads.synth import as_f64

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402

# log2 of a row's largest weight per key block, against block 0, for rows with full slope
PROFILES = {"flat": lambda b, n: 0, "slow": lambda b, n: 6 * b, "fast": lambda b, n: 25 * b, "jump": lambda b, n: 40 * (b >= n // 2),
            "late": lambda b, n: 60 * (b == n - 1), "beyond": lambda b, n: 200 * (b == n // 2), "fall": lambda b, n: -200 * b}


@pytest.mark.parametrize("profile", list(PROFILES))
@pytest.mark.parametrize("d,B,T,H,W,n_text", [(128, 128, 1, 9, 141, 0), (64, 128, 1, 8, 128, 30), (128, 64, 1, 7, 61, 0), (64, 64, 3, 5, 47, 64)])
def test_rows_that_outgrow_their_reference(profile, d, B, T, H, W, n_text):
    print(f"reference {profile} d={d} B={B} {T}x{H}x{W}+{n_text}", flush=True)
    g = P.Geom(T, H, W, n_text, 2, d, B, B // 4)
    s = P.dfs_geom_sizes(g)
    rng = np.random.default_rng(5)
    perm_pad, inv, blk_valid = G.gpu_perm(g)
    valid = blk_valid.cpu().numpy()
    q, k, v = (rng.standard_normal((2, s.N_pad, d)).astype(np.float32) for _ in range(3))
    # feature 0 carries the profile: rows of slope 0, 1/2 and 1, keys at the level of their block
    block = np.arange(s.N_pad) // B
    q[:, :, 0] = 8.0 * (np.arange(s.N_pad) % 3) / 2
    level = np.array([PROFILES[profile](int(b), s.M) for b in range(s.M)], dtype=np.float64)
    k[:, :, 0] = level[block] * math.sqrt(d) / (8.0 * math.log2(math.e))
    pad = np.concatenate([np.arange(B) >= valid[b] for b in range(s.M)])
    for x in (q, k, v):
        x[:, pad] = 0.0
    q, k, v = (to_bf16_bits(x) for x in (q, k, v))
    mask = np.ones((2, s.M, s.M), dtype=np.uint8)
    mask[1, :, 1::3] = 0                                             # head 1: lists of unequal start and stride
    mask[1, :, s.M // 2] = 1
    st = G.upload_mask(mask, s.M)
    dev = [G.to_dev(x) for x in (q, k, v)]
    o, lse = G.gpu_attn(g, P.DFS_BF16, *dev, st)
    o_plain, _ = G.gpu_attn(g, P.DFS_BF16, *dev, st, want_lse=False)
    torch.cuda.synchronize()
    rows = ~pad
    assert torch.equal(o[:, torch.from_numpy(rows).cuda()].view(torch.int16), o_plain[:, torch.from_numpy(rows).cuda()].view(torch.int16))
    got, got_lse = G.as_f64_dev(o), lse.cpu().numpy().astype(np.float64)
    for h in range(2):
        qh, kh, vh = (as_f64(x[h]) for x in (q, k, v))
        for u in range(s.M):
            want, want_lse = O.sparse_attn_block(qh, kh, vh, np.nonzero(mask[h, u])[0], valid, B, u, 1.0 / math.sqrt(d))
            r = slice(u * B, u * B + valid[u])
            err = np.abs(got[h, r] - want[:valid[u]])
            # the path's bf16 bounds; log-sum-exp 1e-4 plus the fp32 rounding of the logits themselves (d products of
            # magnitude up to |logit|, each good to 2^-24, and the change of base)
            assert err.max() <= 2e-2 and err.mean() <= 2e-3, (h, u, err.max(), err.mean())
            bound = 1e-4 + 2.0 ** -20 * np.abs(want_lse[:valid[u]]).max()
            assert np.abs(got_lse[h, r] - want_lse[:valid[u]]).max() <= bound, (h, u)


def _dense(g, q, k, v, want_lse=False):
    """Every block kept; the geometries below have no pad rows."""
    s = P.dfs_geom_sizes(g)
    st = G.upload_mask(np.ones((g.heads, s.M, s.M), dtype=np.uint8), 4)
    return G.gpu_attn(g, P.DFS_BF16, q, k, v, st, want_lse=want_lse)


def _rel(a, b):
    return float((a.double() - b).norm() / b.norm())


SHAPES = [(64, 64), (64, 128), (128, 64), (128, 128)]


@pytest.mark.parametrize("d,B", SHAPES)
@pytest.mark.parametrize("heads,spread", [(1, 2.0), (12, 2.0), (1, 3.0)])
def test_weights_are_exact_where_they_are_largest(d, B, heads, spread):
    """The rounding of the weights to bf16 is against a reference that follows the row: the outputs' error against 64
    bits stays with that of weights rounded against a maximum followed within 2^6 (2 % for the other roundings; a
    reference that stays at the first half tile's maximum is 4 to 5 % above)."""
    g = P.Geom(1, 32, 128, 0, heads, d, B, B // 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + B)
    q, k, v = (torch.randn(heads, 4096, d, generator=gen, device="cuda") for _ in range(3))
    q, k, v = q.bfloat16(), (spread * k).bfloat16(), v.bfloat16()
    got = _dense(g, q, k, v)[0]
    err = norm = err_follow = 0.0
    for h in range(min(heads, 2)):
        x = q[h].double() @ k[h].double().t().contiguous() * (math.log2(math.e) / math.sqrt(d))
        vh = v[h].double()
        want = torch.softmax(x * math.log(2.0), -1) @ vh
        top, ref, weights = x.max(1, keepdim=True).values, x[:, :32].max(1, keepdim=True).values, []
        for i in range(0, 4096, 32):
            high = x[:, i:i + 32].max(1, keepdim=True).values
            ref = torch.where(high - ref > 6, high, ref)
            weights.append(torch.exp2(x[:, i:i + 32] - ref).bfloat16().double() * torch.exp2(ref - top))
        w = torch.cat(weights, 1)
        follow = (w @ vh / w.sum(1, keepdim=True)).bfloat16().double()
        err += float((got[h].double() - want).square().sum())
        err_follow += float((follow - want).square().sum())
        norm += float(want.square().sum())
    print(f"d={d} B={B} heads={heads} spread={spread}: {math.sqrt(err / norm):.4e}, followed within 2^6 {math.sqrt(err_follow / norm):.4e}", flush=True)
    assert err <= 1.02 ** 2 * err_follow


@pytest.mark.parametrize("d,B", SHAPES)
def test_rows_without_a_finite_logit_are_zero(d, B):
    g = P.Geom(1, 1, 3 * B, 0, 2, d, B, B // 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    q, k, v = (torch.randn(2, 3 * B, d, generator=gen, device="cuda").bfloat16() for _ in range(3))
    k = k.abs()
    q[:, 7] = -3e38                                       # logits of -inf with every key
    want = torch.softmax(q.double() @ k.double().transpose(1, 2).contiguous() / math.sqrt(d), -1) @ v.double()
    rows = torch.arange(3 * B, device="cuda") != 7
    for want_lse in (True, False):
        o, lse = _dense(g, q, k, v, want_lse)
        assert not o[:, 7].any() and (not want_lse or bool(torch.isneginf(lse[:, 7]).all()))
        assert _rel(o[:, rows], want[:, rows]) <= 7.5e-3   # the suite's bound for bf16 outputs, relative


@pytest.mark.parametrize("d,B", SHAPES)
@pytest.mark.parametrize("jump", [20, 40, 60, 90])
def test_large_values_under_steep_logits(d, B, jump):
    """Weights stay near one however far a row's logits rise, so values of 2^100 do not overflow the sums."""
    g = P.Geom(1, 1, 3 * B, 0, 1, d, B, B // 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(jump)
    q, k, v = (torch.randn(1, 3 * B, d, generator=gen, device="cuda") for _ in range(3))
    q[:, :, 0] = 8.0
    k[:, :, 0] = (torch.arange(3 * B, device="cuda") // B == 1) * jump * math.sqrt(d) / (8 * math.log2(math.e))
    q, k, v = q.bfloat16(), k.bfloat16(), (v * 2.0 ** 100).bfloat16()
    want = torch.softmax(q.double() @ k.double().transpose(1, 2).contiguous() / math.sqrt(d), -1) @ v.double()
    assert _rel(_dense(g, q, k, v)[0], want) <= 7.5e-3


@pytest.mark.parametrize("d,B", SHAPES)
@pytest.mark.parametrize("heads", [1, 200])              # shared by wave groups or not; above 512 work-groups, one buffer each at (128, 64)
@pytest.mark.parametrize("jump", [140, 200, 1000])
def test_weights_that_overflow_in_every_row_at_once(d, B, heads, jump):
    """A key block so far above the reference that all rows of a wave reach infinite weights in the same half tile: the row sums
    multiply the weights of rows n and n + 16 by zeros of one another's, so that both come out as NaN, and the half tile has
    to be done again all the same."""
    g = P.Geom(1, 1, 3 * B, 0, heads, d, B, B // 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(jump)
    q, k, v = (torch.randn(1, 3 * B, d, generator=gen, device="cuda") for _ in range(3))
    q[:, :, 0] = 8.0
    k[:, :, 0] = (torch.arange(3 * B, device="cuda") // B == 1) * jump * math.sqrt(d) / (8 * math.log2(math.e))
    rows = torch.arange(3 * B, device="cuda") // B != 1  # the others' own block, where their reference starts, is the high one
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    logits = q[0].double() @ k[0].double().t().contiguous() / math.sqrt(d)
    want, want_lse = torch.softmax(logits, -1) @ v[0].double(), torch.logsumexp(logits, -1)
    q, k, v = (x.expand(heads, -1, -1).contiguous() for x in (q, k, v))
    for with_lse in (True, False):
        o, lse = _dense(g, q, k, v, with_lse)
        for r in (rows, ~rows):
            assert _rel(o[:, r], want[r].expand(heads, -1, -1)) <= 7.5e-3
        if with_lse:                                       # the bound of the first test
            assert float((lse.double() - want_lse).abs().max()) <= 1e-4 + 2.0 ** -20 * float(want_lse.abs().max())


@pytest.mark.parametrize("jump", [140, 1000])
def test_weights_that_overflow_where_the_last_round_is_shared(jump):
    """As above through dfs_forward, 520 query blocks: eight of them are shared by several work-groups."""
    g = P.Geom(5, 16, 64, 0, 13, 128, 128, 32)
    s = P.dfs_geom_sizes(g)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(jump)
    q, k, v = (torch.randn(13, s.N, 128, generator=gen, device="cuda") for _ in range(3))
    perm_pad, inv, _ = G.gpu_perm(g)
    q[:, :, 0] = 8.0
    k[:, :, 0] = (inv // 128 % 20 == 11) * jump * math.sqrt(128) / (8 * math.log2(math.e))
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    st = P.MaskState(torch.zeros((13, s.M, s.M), dtype=torch.int32, device="cuda"), torch.full((13, s.M), s.M, dtype=torch.int32, device="cuda"),
                     None, None, s.M)                      # K_max = M: three work-groups to each of the eight
    o = torch.full_like(q, 7.0)
    P.dfs_forward(g, P.DFS_BF16, q, k, v, perm_pad, inv, False, P.DFS_SELECT_TOPK, 0.5, 0.0, st, 128 ** -0.5, o,
                  G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_FORWARD_BF16)))
    for h in range(13):
        want = torch.softmax(q[h].double() @ k[h].double().t().contiguous() * 128 ** -0.5, -1) @ v[h].double()
        assert _rel(o[h], want) <= 7.5e-3


@pytest.mark.parametrize("d,B,below", [(64, 64, 20), (64, 64, 22), (64, 128, 19), (64, 128, 21), (128, 64, 20), (128, 64, 22), (128, 128, 19), (128, 128, 21)])
def test_small_weights_behind_large_ones_are_counted(d, B, below):
    """131 072 keys, those behind the first block 2^-below as heavy: each half tile of them weighs about as much as the last
    place of the row's sum.  Only the first block has values, so that the outputs are inverse to the row sums.  4 096 half
    tiles, each added with an error of half a last place, 2^-24 of the sum, at most; the outputs' own rounding averages out
    over 8 192 rows."""
    N = 131072
    g = P.Geom(1, 256, 512, 0, 1, d, B, B // 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(below)
    q, k = (0.3 * torch.randn(1, N, d, generator=gen, device="cuda") for _ in range(2))
    q[:, :, 0] = 8.0
    k[:, :, 0] = 0.0
    k[:, B:, 0] = -below * math.sqrt(d) / (8 * math.log2(math.e))
    v = 1 + torch.rand(1, N, d, generator=gen, device="cuda")
    v[:, B:] = 0.0
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    kd, vd = k[0].double().t().contiguous(), v[0].double()
    want = torch.cat([torch.softmax(x.double() @ kd / math.sqrt(d), -1) @ vd for x in q[0, :8192].split(2048)])
    cnt = torch.full((1, N // B), N // B, dtype=torch.int32, device="cuda")
    st = P.MaskState(torch.zeros((1, N // B, 1), dtype=torch.int32, device="cuda"), cnt, None, None, 1)
    for with_lse in (False, True):
        o = G.gpu_attn(g, P.DFS_BF16, q, k, v, st, want_lse=with_lse)[0]
        off = float((o[0, :8192].double() / want - 1).mean())
        print(f"d={d} B={B} below={below} lse={with_lse}: {off:+.2e}", flush=True)
        assert abs(off) <= 4096 * 2.0 ** -24
