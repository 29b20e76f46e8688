"""Selection of a row at the lengths where its way changes (ranked outright, keys in registers, histogram): rows full of ties, of zeros of both signs,
negative and very small scores, and a keep count from one to all, against an ordering on the host."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from tests import gpu_util as G  # noqa: E402


@pytest.mark.parametrize("M_v", [1, 3, 16, 17, 63, 64, 65, 128, 192, 193, 320, 321, 448, 449, 640, 641, 900])
def test_rows_of_every_length(M_v):
    H, W = next((n // w, w) for n in range(M_v * 64, (M_v - 1) * 64, -1) for w in range(512, 0, -1) if n % w == 0 and n // w <= 512)
    g = P.Geom(1, H, W, 70, 2, 64, 64, 16)
    s = P.dfs_geom_sizes(g)
    assert s.M_v == M_v
    rng = np.random.default_rng(M_v)
    score = rng.random((2, M_v, M_v), dtype=np.float32)
    kind = np.arange(M_v) % 6
    score[:, kind == 1] = rng.integers(0, 3, (2, (kind == 1).sum(), M_v)).astype(np.float32)              # ties
    score[:, kind == 2] = np.where(rng.random((2, (kind == 2).sum(), M_v)) < 0.5, 0.0, -0.0)               # they rank alike
    score[:, kind == 3] -= 0.5
    score[:, kind == 4] *= np.float32(1e-42)                                                              # subnormal
    score[:, kind == 5] = np.float32(2.0) ** rng.integers(-120, 120, (2, (kind == 5).sum(), M_v))
    dev = torch.from_numpy(score).cuda()
    for k in sorted({1, (M_v + 2) // 3, M_v - 1, M_v} - {0}):
        st = G.gpu_select(g, dev, P.DFS_SELECT_TOPK, 1 - k / M_v)
        assert P.dfs_keep_count(1 - k / M_v, M_v) == k
        order = np.argsort(-score, axis=-1, kind="stable")[:, :, :k]                                      # equal scores: the lower column first
        want = np.sort(order, axis=-1)
        idx = st.kv_idx.cpu().numpy()[:, :M_v]
        assert np.array_equal(idx[:, :, :k], want)
        assert np.array_equal(idx[:, :, k:k + s.M_x], np.broadcast_to(np.arange(M_v, s.M), (2, M_v, s.M_x)))
        mask = np.zeros((2, M_v, s.M), dtype=np.uint8)
        np.put_along_axis(mask, want, 1, axis=-1)
        mask[:, :, M_v:] = 1
        assert np.array_equal(st.mask.cpu().numpy()[:, :M_v], mask)
        assert (st.kv_cnt.cpu().numpy()[:, :M_v] == k + s.M_x).all()
