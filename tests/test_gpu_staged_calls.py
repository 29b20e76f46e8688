"""The staged calls of a quality check take plain arguments without marshalling in Python (_calls).  What is not plain goes the other way: the same
results where it was accepted, the same error where it was not."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2605_23445_amd")
from paper_2605_23445_amd import _calls  # noqa: E402
from tests import gpu_util as G  # noqa: E402


def _calls_of(dtype):
    """Name, native function, arguments by name, the outputs among them."""
    g = P.Geom(2, 6, 11, 5, 2, 64, 64, 16)
    s = P.dfs_geom_sizes(g)
    td = torch.bfloat16 if dtype == P.DFS_BF16 else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.randn(2, s.N, 64, generator=gen, device="cuda").to(td)
    q, k, v = (torch.randn(2, s.N_pad, 64, generator=gen, device="cuda").to(td) for _ in range(3))
    perm_pad, inv, _ = G.gpu_perm(g)
    i32 = dict(dtype=torch.int32, device="cuda")
    score = torch.rand(2, s.M_v, s.M_v, generator=gen, device="cuda")
    idx, cnt = torch.zeros((2, s.M, s.M), **i32), torch.full((2, s.M), s.M, **i32)
    lse = torch.randn(2, 2, s.N_pad, generator=gen, device="cuda")
    ws = G.ws_tensor(max(P.dfs_workspace_bytes(g, kind) for kind in (P.DFS_WS_BLOCK_SCORE, P.DFS_WS_SELECT_MASK)))
    new = lambda *shape, t=td: torch.zeros(shape, dtype=t, device="cuda")  # noqa: E731
    return [
        (P.dfs_permute, _calls.permute, dict(g=g, dtype=dtype, x=x, perm_pad=perm_pad, x_perm=new(2, s.N_pad, 64)), ["x_perm"]),
        (P.dfs_unperm, _calls.unperm, dict(g=g, dtype=dtype, o_perm=q, inv=inv, o=new(2, s.N, 64)), ["o"]),
        (P.dfs_block_score, _calls.block_score, dict(g=g, dtype=dtype, q_perm=q, k_perm=k, score=new(2, s.M_v, s.M_v, t=torch.float32), ws=ws), ["score"]),
        (P.dfs_select_mask, _calls.select_mask, dict(g=g, score=score, mode=P.DFS_SELECT_MASS_HEAD, sparsity=0.9, mass=0.6, mask=new(2, s.M, s.M, t=torch.uint8),
                                                     kv_idx=new(2, s.M, s.M, t=torch.int32), kv_cnt=new(2, s.M, t=torch.int32), K_max=s.M,
                                                     k_head=new(2, t=torch.int32), ws=ws), ["mask", "kv_cnt", "k_head"]),
        (P.dfs_sparse_attn_fwd, _calls.sparse_attn, dict(g=g, dtype=dtype, q_perm=q, k_perm=k, v_perm=v, kv_idx=idx, kv_cnt=cnt, K_max=s.M, scale=0.125,
                                                         o_perm=new(2, s.N_pad, 64), lse=new(2, s.N_pad, t=torch.float32)), ["o_perm", "lse"]),
        (P.dfs_recall, _calls.recall, dict(g=g, lse_sparse=lse[0], lse_dense=lse[1], recall=new(2, t=torch.float32)), ["recall"]),
    ]


class _Tensor(torch.Tensor):
    pass


@pytest.mark.parametrize("dtype", [P.DFS_BF16, P.DFS_F32])
@pytest.mark.parametrize("i", range(6))
def test_same_either_way(i, dtype):
    call, native, args, outs = _calls_of(dtype)[i]
    assert native(*args.values()) == 0
    want = {name: args[name].clone() for name in outs}
    changes = [{name: args[name].as_subclass(_Tensor)} for name in args if isinstance(args[name], torch.Tensor)]
    changes += [{name: np.float64(args[name])} for name in args if isinstance(args[name], float)] + [{}]
    for change in changes:
        a = dict(args, **change)
        for name in outs:
            args[name].fill_(7)                            # the changed argument has its memory
        assert (native(*a.values()) is None) == bool(change), change.keys()
        for name in outs:
            args[name].fill_(7)
        call(**a)
        for name in outs:
            assert torch.equal(args[name], want[name]), (name, change.keys())
    for name in ("mask", "k_head", "lse"):                 # where None is taken
        if name in args:
            assert native(*dict(args, **{name: None}).values()) == 0
            call(**dict(args, **{name: None}))


@pytest.mark.parametrize("i", range(6))
def test_what_was_refused_is_refused(i):
    call, native, args, _ = _calls_of(P.DFS_BF16)[i]
    for name, x in args.items():
        if not isinstance(x, torch.Tensor):
            continue
        bad = [x.cpu(), x.reshape(-1)[: x.numel() // 2] if name != "ws" else x[:256]] + ([x.half()] if name != "ws" else [])
        if x.dim() > 1:
            bad.append(x.transpose(0, 1))
        for b in bad:
            a = dict(args, **{name: b})
            assert native(*a.values()) != 0
            with pytest.raises((ValueError, P.DfsError)):
                call(**a)
        if name not in ("mask", "k_head", "lse"):
            a = dict(args, **{name: None})
            assert native(*a.values()) != 0
            with pytest.raises(P.DfsError):
                call(**a)
    bad = {"g": P.Geom(2, 6, 11, 5, 2, 96, 64, 16), "dtype": 5, "mode": 7, "sparsity": 1.5, "K_max": 0, "scale": -1.0}
    for name in set(bad) & set(args):
        with pytest.raises((ValueError, P.DfsError)):
            call(**dict(args, **{name: bad[name]}))
