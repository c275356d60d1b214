"""Selection where a launch takes another turn: rows around the lengths that one register or one more per lane holds, without
slack vouched for behind the array (the last rows then read other columns; a single row is all last); and the whole-map histograms
with one to eight chunks of a map per workgroup.  Scores with many ties, infinities and NaN.  Against the oracle."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from gpu_util import say

pytestmark = pytest.mark.gpu


def _scores(H, g, seed):
    rng = np.random.default_rng(seed)
    L = (rng.normal(size=(1, H, g, g)) * 4).astype(np.float32)
    L[0, :, :, ::3] = np.round(L[0, :, :, ::3])
    for value in (np.inf, -np.inf, np.nan, -0.0):
        L[0, rng.integers(H, size=g), rng.integers(g, size=g), rng.integers(g, size=g)] = value
    return L


@pytest.mark.parametrize("g", [1, 2, 63, 64, 65, 1000, 1024, 1025, 2047, 2048, 2049, 4000, 4096])
def test_rows(g):
    import torch
    L = _scores(1, g, g)
    for keep in sorted({1, max(1, g // 7), g}):
        say(f"select rows {g} keep {keep}")
        p = da.problem(1, 1, g, 8, 8, 128, 8, 8, keep_blocks=keep)
        idx = torch.full((1, 1, g, keep), -1, dtype=torch.int32, device="cuda")
        mask = torch.full((1, 1, g, g), 9, dtype=torch.uint8, device="cuda")
        da.da_select_blocks(p, torch.from_numpy(L).cuda(), idx, mask)
        torch.cuda.synchronize()
        want_idx, want_mask = oa.select_blocks(L[0, 0], keep)[:2]
        assert np.array_equal(idx[0, 0].cpu().numpy(), want_idx)
        assert np.array_equal(mask[0, 0].cpu().numpy(), want_mask)


@pytest.mark.parametrize("g,H", [(600, 1), (600, 24), (450, 64), (301, 130), (700, 80)])   # 1, 2, 3, 2 (a short last one), 8 chunks
def test_whole_map_groups(g, H):
    import torch
    say(f"whole map {H} x {g}")
    L = _scores(H, g, H)
    p = da.problem(1, H, g, 8, 8, 128, 8, 8, sparsity=0.9)
    sz = da.da_global_sizes(p)
    row_ptr = torch.full((1, H, g + 1), -1, dtype=torch.int32, device="cuda")
    cols = torch.full((1, H, sz.cap), -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(sz.select_ws, dtype=torch.uint8, device="cuda")
    da.da_select_blocks_global(p, torch.from_numpy(L).cuda(), row_ptr, cols, ws, None)
    torch.cuda.synchronize()
    rp, cl = row_ptr.cpu().numpy(), cols.cpu().numpy()
    for h in range(0, H, max(1, H // 6)):
        want_rp, want_cols = oa.select_blocks_global(L[0, h], sz.budget)[:2]
        assert np.array_equal(rp[0, h], want_rp)
        assert np.array_equal(cl[0, h, :want_rp[-1]], want_cols)
