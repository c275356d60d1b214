"""The tile counts of da_sparse_attn_ex follow what is worked on: tiles of which the first or the last 32 keys are negligible
count half in the second number, tiles with at most 32 valid keys count whole when they are carried out, and query tiles
that hold nothing but pad slots count nowhere."""
import numpy as np
import pytest

from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import empty, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pw", [8, 16])
@pytest.mark.parametrize("best", ["first", "last", "both"])
@pytest.mark.parametrize("T,fh,fw", [(1, 8, 16), (4, 8, 16), (66, 16, 16), (5, 8, 48), (4, 8, 20)])
def test_half_dropped_tiles(T, fh, fw, best, pw):
    import torch
    say(f"tile counts {T}x{fh}x{fw} window 8x{pw} {best}")
    n = T * fh * fw
    rng = np.random.default_rng(fw)
    Q, K, V = rng.normal(size=(3, 1, 1, n, 128)) * 0.1
    p = da.problem(1, 1, T, fh, fw, 128, 8, pw)
    dims = da.da_derive(p)
    perm = torch.empty(dims.n_pad, dtype=torch.int32, device="cuda")
    valid = torch.empty(dims.g, dtype=torch.int32, device="cuda")
    da.da_build_perm(p, perm, None, valid)
    # scores of one half of each 64 slots lie some 130 powers of two above the other half's (a tile of at most 32 keys is
    # all first half)
    slot = np.empty(n, np.int64)
    tokens = perm.cpu().numpy()
    slot[tokens[tokens >= 0]] = np.nonzero(tokens >= 0)[0] % 64
    sub_valid = np.clip(valid.cpu().numpy()[:, None] - np.arange(0, dims.block, 64), 0, 64)      # valid keys of each tile
    Q[..., 0], K[..., 0] = 32.0, 0.0
    if best != "both":
        K[..., 0] = np.where((slot < 32) == (best == "first"), 16.0, -16.0)
    x = [to_dev(W.to_storage(a, W.BF16), W.BF16) for a in (Q, K, V)]
    Kp = empty((1, 1, dims.n_pad, 128), W.BF16)
    Vt, O = torch.empty_like(Kp), empty((1, 1, n, 128), W.BF16)
    da.da_permute(p, x[1], Kp, da.DA_REORDER_ROWS)
    da.da_permute(p, x[2], Vt, da.DA_REORDER_VOP)
    idx = torch.arange(dims.g, dtype=torch.int32, device="cuda").repeat(dims.g, 1).contiguous()
    counts = torch.zeros(2, dtype=torch.int64, device="cuda")
    da.da_sparse_attn_ex(p, x[0], Kp, Vt, idx, O, None, 1, counts)
    torch.cuda.synchronize()
    seen, kept = (int(c) for c in counts.cpu())
    query_tiles = int(np.ceil(valid.cpu().numpy() / 32).sum())
    tiles, short = int((sub_valid > 0).sum()), int(((sub_valid > 0) & (sub_valid <= 32)).sum())
    assert seen == query_tiles * tiles
    if best == "both":
        assert kept == seen
    elif best == "first":
        # rounded to whole tiles once per wave with 32 queries: at most eight waves share a list
        narrow = int((sub_valid > 0).sum() * 2 - query_tiles)
        assert abs(kept - query_tiles * (short + 0.5 * (tiles - short))) <= 4 * narrow
    else:
        # what a wave meets first is carried out, whatever it is worth
        assert query_tiles * 0.5 * (tiles - short) - 8 * tiles <= kept <= query_tiles * (0.5 * (tiles - short) + 8)
        assert kept < seen or tiles <= 8


def test_odd_counts_are_rounded_evenly():
    """Seven frames of 8x12: blocks of 64 and of 32 valid slots, 200 units of one wave per list.  A wave with 32 queries carries out half
    of each of seven whole tiles and seven short ones: its count is 10.5, and 700 such waves are to round up about as often as down (of the seven of a head one more)."""
    import torch
    say("tile counts, odd counts of one wave per list")
    T, fh, fw, H = 7, 8, 12, 100
    p = da.problem(1, H, T, fh, fw, 128, 8, 8)
    dims = da.da_derive(p)
    n = T * fh * fw
    perm = torch.empty(dims.n_pad, dtype=torch.int32, device="cuda")
    da.da_build_perm(p, perm, None, None)
    tokens = perm.cpu().numpy()
    slot = np.empty(n, np.int64)
    slot[tokens[tokens >= 0]] = np.nonzero(tokens >= 0)[0] % 64
    Q = np.zeros((1, H, n, 128))
    K = np.zeros_like(Q)
    Q[..., 0], K[..., 0] = 32.0, np.where(slot < 32, 16.0, -16.0)
    q, k = (to_dev(W.to_storage(a, W.BF16), W.BF16) for a in (Q, K))
    Kp = empty((1, H, dims.n_pad, 128), W.BF16)
    Vt, O = torch.empty_like(Kp), empty((1, H, n, 128), W.BF16)
    da.da_permute(p, k, Kp, da.DA_REORDER_ROWS)
    da.da_permute(p, k, Vt, da.DA_REORDER_VOP)
    idx = torch.arange(dims.g, dtype=torch.int32, device="cuda").repeat(H * dims.g, 1).contiguous()
    counts = torch.zeros(2, dtype=torch.int64, device="cuda")
    da.da_sparse_attn_ex(p, q, Kp, Vt, idx, O, None, 1, counts)
    torch.cuda.synchronize()
    seen, kept = (int(c) for c in counts.cpu())
    assert seen == H * T * (2 + 1) * 2 * T
    exact = H * T * 3 * (7 * 0.5 + 7)
    say(f"  carried out {kept}, exactly {exact}")
    assert abs(kept - exact) <= 0.1 * H * T
