"""Which kernels a call launches and with what grids, recorded on the CPU with a stand-in for the HIP runtime's launch functions."""
import os

import pytest

from paper_2505_14708_amd import binding as da
from launch_recorder import record

pytestmark = pytest.mark.skipif(not os.path.exists(da.LIB_PATH), reason="library not built")


def _problem(B, H, T, fh, fw, keep, *, d=128, pw=8, dtype=da.DA_BF16):
    return dict(B=B, H=H, T=T, fh=fh, fw=fw, d=d, ph=8, pw=pw, dtype=dtype, keep_blocks=keep, sparsity=0.0, pool=0, reserved=0)


def test_grids_stay_within_the_launch_limits(tmp_path):
    """A launch has fewer than 2^32 threads along each axis and at most 65535 workgroups along y and z.  Frames that are
    mostly padding make many blocks of few tokens: 7500 heads of 100 frames of 1x57 tokens are six million blocks, 200 GB of reordered K
    and V beside 44 GB of Q, K, V and O, which a card with 288 GB holds."""
    calls = [(e, _problem(1, 7500, 100, 1, 57, k)) for e in ("da_forward", "da_forward_global") for k in (1, 320, 800)]
    calls += [(e, _problem(1, 60000, 100, 1, 1, k)) for e in ("da_forward", "da_forward_blocks", "da_forward_global") for k in (1, 40, 100)]
    calls += [(e, _problem(1, 3, 1700, 9, 9, k)) for e in ("da_forward", "da_forward_global") for k in (1, 600, 6800)]
    for (entry, p), (status, launches) in zip(calls, record(str(tmp_path), calls)):
        assert status == da.DA_OK and launches, (entry, p)
        for name, grid, group, lds in launches:
            assert all(0 < n * g < 1 << 32 for n, g in zip(grid, group)), (name, grid, group, p)
            assert max(grid[1:]) <= 65535, (name, grid)


@pytest.mark.parametrize("dtype,d", [(da.DA_BF16, 128), (da.DA_F32, 64)])
def test_logits_and_lists_in_one_launch(tmp_path, dtype, d):
    """Where a map's rows have at most 64 columns and there are at most two workgroups (of 32 rows) for every CU, or a workgroup has
    at least 16 of its rows and the map no more."""
    cases = [(B * 24, g) for B in (1, 5, 11, 21, 22, 64) for g in (2, 15, 16, 28, 32, 33, 64, 65)]
    calls = [("da_forward", _problem(1, H, g, 8, 8, 1, d=d, dtype=dtype)) for H, g in cases]
    for (H, g), (status, launches) in zip(cases, record(str(tmp_path), calls)):
        assert status == da.DA_OK
        names = " ".join(l[0] for l in launches)
        one = g <= 64 and (H * -(-g // 32) <= 512 or 16 <= g <= 32)
        assert ("draft_select_kernel" in names, "draft_logits_kernel" in names) == (one, not one), (H, g)


def test_float32_last_rounds_in_pieces(tmp_path):
    """One head of 28 frames of 39x45 tokens: 210 half blocks to an XCD, all of which hold queries, 64 at a time.  The last 18 are cut in
    two only where lists are of any length."""
    p = _problem(1, 1, 28, 39, 45, 84, dtype=da.DA_F32)
    grids = [[g for name, g, _, _ in launches if "attn_f32" in name][0][0] for _, launches in
             record(str(tmp_path), [("da_forward", p), ("da_forward_global", p), ("da_forward", dict(p, keep_blocks=840))])]
    assert grids == [8 * 210, 8 * (192 + 2 * 18), 8 * 210]
