"""bf16 attention when a row's logits outgrow the reference its softmax started with: rows that grow slowly (the
reference moves along), in jumps, beyond what a sum can hold (the block is done again from the true maximum), only in
the last block, and rows that fall.  Against the oracle under the same lists, through the C ABI."""
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
