"""Token orders, bit-exact against the oracle, on grids where the clipped extents of the sub-cubes can go wrong: axes of one
cell, of the largest extent, of a power of two and one beside it."""
import numpy as np
import pytest
import torch

from oracle import dfs_oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("T,H,W,n_text", [(1, 1, 512, 0), (512, 1, 3, 5), (2, 512, 2, 0), (1, 2, 1, 1), (2, 2, 2, 0), (8, 8, 8, 0),
                                          (7, 9, 8, 0), (9, 7, 17, 64), (15, 16, 17, 3), (5, 257, 3, 0), (31, 33, 1, 130)])
def test_token_orders_on_edge_grids(T, H, W, n_text):
    g = P.Geom(T, H, W, n_text, 1, 64, 64, 64)
    s = P.dfs_geom_sizes(g)
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_HILBERT_PERM))
    for kind, order in (("hilbert3d", P.DFS_ORDER_HILBERT3D), ("raster", P.DFS_ORDER_RASTER),
                        ("hilbert2d", P.DFS_ORDER_HILBERT2D), ("block3d", P.DFS_ORDER_BLOCK3D)):
        out = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (s.N_pad, s.N, s.M)]
        P.dfs_token_order(g, order, *out, ws)
        for got, want in zip(out, O.token_order(kind, T, H, W, n_text, 64)):
            assert np.array_equal(got.cpu().numpy(), want), kind


@pytest.mark.parametrize("T,H,W", [(512, 32, 512), (509, 32, 511), (31, 512, 512), (200, 200, 200), (1, 512, 509)])
def test_token_order_on_the_largest_grids(T, H, W):
    """Up to 2^23 tokens (65 536 blocks), whose numbers the kernel divides by the extents: the order and its inverse fit together, and
    the Hilbert indices of the oracle ascend along it (at 2^16 positions)."""
    g = P.Geom(T, H, W, 0, 1, 64, 128, 128)
    s = P.dfs_geom_sizes(g)
    ws = G.ws_tensor(P.dfs_workspace_bytes(g, P.DFS_WS_HILBERT_PERM))
    perm, inv, valid = (torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (s.N_pad, s.N, s.M))
    P.dfs_token_order(g, P.DFS_ORDER_HILBERT3D, perm, inv, valid, ws)
    assert torch.equal(perm[inv.long()], torch.arange(s.N, dtype=torch.int32, device="cuda"))
    at = np.unique(np.random.default_rng(T).integers(0, s.N, 2 ** 16))
    n = perm.cpu().numpy()[at].astype(np.int64)
    key = O.hilbert_key(n // (H * W), n // W % H, n % W, O.cube_bits(T, H, W))
    assert np.all(np.diff(key) > 0)
