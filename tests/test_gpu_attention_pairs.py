"""The bf16 attention where the waves of a query block can divide its list wrongly: lists of one entry (all waves but one get
none), of odd and even length, and of every block; blocks with at most 32 valid slots (half a tile, one wave's worth of queries);
frame counts that leave one to seven frames over.  One head, whose units are each shared by eight workgroups (eight waves to a list),
and as many heads as it takes for four, two and one wave to a list, alone and together in one launch, each around the
lengths at which its waves begin to do otherwise: eight tiles to each wave (all look at their own block first), and 24 where there is one wave.
As generated (most tiles dropped) and with Q scaled down (none).  Against the oracle, within the build target's bounds for
bf16 outputs."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, TOL, empty, output_error, say, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


# (T, fh, fw, pw, heads, how many workgroups share a unit: 2^..., one number for all or for the first and the last units): kept blocks
SHARED = {(9, 20, 24, 8, 1, (3,)): (7, 9, 63, 64, 65, 81), (4, 20, 40, 16, 1, (3,)): (31, 32, 33),
          (5, 12, 28, 8, 9, (2,)): (1, 3, 5, 31, 32, 33, 40), (3, 20, 40, 16, 9, (2,)): (1, 15, 16, 17, 27),
          (5, 12, 28, 8, 20, (1,)): (1, 2, 3, 15, 16, 17, 40), (3, 20, 40, 16, 18, (1,)): (1, 7, 8, 9, 27),
          (5, 12, 28, 8, 40, (0,)): (1, 2, 7, 8, 9, 23, 24, 25, 40), (3, 20, 40, 16, 32, (0,)): (1, 3, 4, 5, 11, 12, 13, 27),
          (5, 12, 28, 8, 52, (0, 2)): (1, 8, 23, 24, 33), (5, 12, 28, 8, 70, (0, 1)): (2, 9, 16, 24),
          (5, 12, 28, 8, 30, (1, 2)): (24, 31, 33), (3, 20, 40, 16, 22, (1, 2)): (12, 15, 17)}


def run(T, fh, fw, pw, H, keep, gain):
    """One forward pass; the first and the last heads against the oracle."""
    import torch
    w = W.Workload("pairs", B=1, H=H, d=128, T=T, fh=fh, fw=fw, pw=pw, seed=fh + T)
    say(f"pairs {T}x{fh}x{fw} window 8x{pw} heads {H} keep {keep} gain {gain}")
    Q, K, V = W.make_qkv(w)
    Q = W.to_storage(W.storage_to_f64(Q, w.dtype) * gain, w.dtype)
    p = da.problem(1, H, T, fh, fw, 128, 8, pw, keep_blocks=keep)
    dims = da.da_derive(p)
    O = empty((1, H, dims.n, 128), w.dtype)
    O.fill_(float("nan"))
    idx = torch.empty((1, H, dims.g, dims.k), dtype=torch.int32, device="cuda")
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    da.da_forward(p, *(to_dev(x, w.dtype) for x in (Q, K, V)), O, ws, idx)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(O).all())
    host, host_idx = to_host_f64(O, w.dtype), idx.cpu().numpy()
    for h in sorted({0, H // 3, H - 2, H - 1} & set(range(H))):
        ref = HeadRef(w, Q[0, h], K[0, h], V[0, h], keep_blocks=keep)
        assert np.array_equal(host_idx[0, h], ref.idx)
        emax, emean = output_error(host[0, h], oa.restore(ref.attention(), ref.inv))
        assert emax <= TOL[w.dtype][0] and emean <= TOL[w.dtype][1], (h, emax, emean)
    assert da.da_wait_failures() == 0


@pytest.mark.parametrize("keep", [1, 2, 3, 15, 16, 17, 34, 10 ** 6])
@pytest.mark.parametrize("T,fh,fw,pw,gain", [(4, 12, 28, 8, 1.0), (5, 12, 28, 8, 0.03125), (7, 20, 19, 8, 1.0), (3, 20, 40, 16, 1.0),
                                             (6, 12, 40, 16, 0.03125)])
def test_lists_of_every_length(T, fh, fw, pw, gain, keep):
    run(T, fh, fw, pw, 1, keep, gain)


@pytest.mark.parametrize("gain", [1.0, 0.03125])
@pytest.mark.parametrize("shape,keep", [(s[:5], k) for s, keeps in SHARED.items() for k in keeps])
def test_lists_of_every_length_by_waves(shape, keep, gain):
    run(*shape, keep, gain)
