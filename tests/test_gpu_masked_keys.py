"""Keys that finite inputs put at a score of minus infinity: one channel of K far below zero marks them, the same channel of Q
is large, and the product leaves the range of float32.  Such keys weigh nothing, wherever they stand: the first or the last
rows of every block, whole blocks, a query's own block, all but one block of a list.  A wave of the attention kernels may
well meet nothing else among its share of the keys.  Against the oracle, whose scores stay finite in float64; tolerances of
the build target (the marked keys contribute exact zeros)."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, TOL, empty, output_error, say, to_dev, to_host_f64

pytestmark = pytest.mark.gpu

# token coordinates -> marked
PATTERNS = {
    "first_rows": lambda t, y, x: y % 8 < 4,
    "last_rows": lambda t, y, x: y % 8 >= 2,
    "first_frame": lambda t, y, x: t == 0,
    "last_frames": lambda t, y, x: t >= 1,
    "left_half": lambda t, y, x: x < 8,
    "all_but_one_block": lambda t, y, x: (t > 0) | (y >= 8) | (x < 8),
}


@pytest.mark.parametrize("pattern", list(PATTERNS))
@pytest.mark.parametrize("dtype,H,T,pw,keep", [(W.F32, 1, 4, 8, 10 ** 6), (W.F32, 1, 4, 8, 3), (W.BF16, 1, 4, 8, 10 ** 6),
                                               (W.BF16, 1, 4, 8, 3), (W.BF16, 1, 18, 8, 10 ** 6), (W.BF16, 1, 4, 16, 10 ** 6),
                                               (W.BF16, 1, 66, 8, 40), (W.BF16, 2, 66, 8, 3)])
def test_masked_keys(dtype, H, T, pw, keep, pattern):
    import torch
    w = W.Workload("masked", B=1, H=H, d=128, T=T, fh=16, fw=32 if pw == 16 else 16, pw=pw, dtype=dtype, seed=T)
    say(f"masked keys dtype {dtype} {H}x{T}x{w.fh}x{w.fw} window 8x{pw} keep {keep} {pattern}")
    Q, K, V = (W.storage_to_f64(x, dtype) for x in W.make_qkv(w))
    t, y, x = np.unravel_index(np.arange(w.N), (T, w.fh, w.fw))
    marked = PATTERNS[pattern](t, y, x)
    assert 0 < marked.sum() < w.N
    Q, K = Q * 0.125, K.copy()
    Q[..., 0] = 2.0 ** 13                                   # products of 2^13 * -2^117: finite inputs, no finite score
    K[..., 0] = np.where(marked, -2.0 ** 117, 0.0)
    Q, K, V = (W.to_storage(a, dtype) for a in (Q, K, V))
    p = da.problem(1, H, T, w.fh, w.fw, 128, 8, pw, dtype=da.DA_F32 if dtype == W.F32 else da.DA_BF16, keep_blocks=keep)
    dims = da.da_derive(p)
    refs = [HeadRef(w, Q[0, h], K[0, h], V[0, h], keep_blocks=keep) for h in range(H)]
    dQ, dK, dV = (to_dev(a, dtype) for a in (Q, K, V))
    O = empty((1, H, dims.n, 128), dtype)
    idx = torch.empty((1, H, dims.g, dims.k), dtype=torch.int32, device="cuda")
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    da.da_forward(p, dQ, dK, dV, O, ws, idx)
    # the stages as well, on lists that begin with the blocks that have the most marked keys
    perm = refs[0].perm
    share = np.where(perm >= 0, marked[np.maximum(perm, 0)], True).reshape(dims.g, dims.block).mean(axis=1)
    host_idx = idx[0].cpu().numpy()
    lists = np.take_along_axis(host_idx, np.argsort(-share[host_idx], axis=2, kind="stable"), axis=2)
    Qp, Kp, Vt, Op = (empty((1, H, dims.n_pad, 128), dtype) for _ in range(4))
    da.da_permute(p, dQ, Qp, da.DA_REORDER_ROWS)
    da.da_permute(p, dK, Kp, da.DA_REORDER_ROWS)
    da.da_permute(p, dV, Vt, da.v_layout(p.dtype))
    lse = torch.empty((1, H, dims.n_pad), dtype=torch.float32, device="cuda")
    da.da_sparse_attn(p, Qp, Kp, Vt, torch.from_numpy(np.ascontiguousarray(lists)).cuda(), Op, lse)
    torch.cuda.synchronize()
    got, got_p, got_lse = to_host_f64(O, dtype)[0], to_host_f64(Op, dtype)[0], lse[0].cpu().numpy()
    for h, ref in enumerate(refs):
        assert np.array_equal(host_idx[h], ref.idx)
        want, want_lse = ref.attention(want_lse=True)
        rows = (perm >= 0) & np.repeat((share[host_idx[h]] < 1.0).any(axis=1), dims.block)   # queries with a key left
        assert rows.any()
        for out in (got[h][perm[rows]], got_p[h][rows]):
            emax, emean = output_error(out, want[rows])
            assert emax <= TOL[dtype][0] and emean <= TOL[dtype][1], (h, emax, emean)
        assert np.abs(got_lse[h][rows] - want_lse[rows]).max() <= (1e-4 if dtype == W.F32 else 2e-2)
    assert da.da_wait_failures() == 0


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_nothing_but_masked_keys(dtype):
    """Rows whose keys all score minus infinity have no softmax and stay NaN; rows without any key at all are zero."""
    import torch
    w = W.Workload("masked_all", B=1, H=1, d=128, T=2, fh=16, fw=16, dtype=dtype, seed=3)
    say(f"all keys masked dtype {dtype}")
    Q, K, V = (W.storage_to_f64(x, dtype) for x in W.make_qkv(w))
    Q[..., 0], K[..., 0] = 2.0 ** 13, -2.0 ** 117
    p = da.problem(1, 1, 2, 16, 16, 128, dtype=da.DA_F32 if dtype == W.F32 else da.DA_BF16)
    dims = da.da_derive(p)
    Qp, Kp, Vt, Op = (empty((1, 1, dims.n_pad, 128), dtype) for _ in range(4))
    da.da_permute(p, to_dev(W.to_storage(Q, dtype), dtype), Qp, da.DA_REORDER_ROWS)
    da.da_permute(p, to_dev(W.to_storage(K, dtype), dtype), Kp, da.DA_REORDER_ROWS)
    da.da_permute(p, to_dev(W.to_storage(V, dtype), dtype), Vt, da.v_layout(p.dtype))
    lengths = np.array([0, 1, 2, 3, 4, 5, 8, 0])
    row_ptr = torch.from_numpy(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)).cuda()
    cols = torch.from_numpy(np.concatenate([np.arange(n) for n in lengths] + [[0]]).astype(np.int32)).cuda()
    da.da_sparse_attn_lists(p, Qp, Kp, Vt, row_ptr, cols, cols.numel(), Op)
    torch.cuda.synchronize()
    got = to_host_f64(Op, dtype)[0, 0].reshape(dims.g, -1)
    assert np.isnan(got[lengths > 0]).all() and (got[lengths == 0] == 0.0).all()
