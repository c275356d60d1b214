"""The bf16 attention where a launch has units that are shared out differently: halves and quarters, whole ones and quarters, whole ones
and halves (in the second and after the fourth round), and where the frames left over make units of blocks of one position or of
several.  Against the oracle on some heads, the first and the last among them, within the build target's bounds for bf16 outputs."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, TOL, empty, output_error, say, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


# (T, fh, fw, pw, heads, kept blocks): the first and the last units are shared by 2^... workgroups each (one number: all alike)
SHARED = {(7, 20, 28, 8, 16, 40): (1, 2), (15, 20, 20, 8, 15, 30): (0,), (9, 20, 28, 8, 23, 17): (0, 1), (8, 18, 20, 8, 116, 9): (0, 1),
          (7, 20, 40, 16, 18, 25): (0, 2), (31, 13, 9, 8, 3, 124): (2,), (1, 13, 9, 8, 1, 3): (3,), (7, 20, 28, 8, 36, 9): (0, 2)}


@pytest.mark.parametrize("gain", [1.0, 0.03125])
@pytest.mark.parametrize("T,fh,fw,pw,H,keep", list(SHARED))
def test_units_shared_out_differently(T, fh, fw, pw, H, keep, gain):
    import torch
    w = W.Workload("units", B=1, H=H, d=128, T=T, fh=fh, fw=fw, pw=pw, seed=fh + T)
    say(f"units {T}x{fh}x{fw} window 8x{pw} heads {H} keep {keep} gain {gain}")
    Q, K, V = W.make_qkv(w)
    Q = W.to_storage(W.storage_to_f64(Q, w.dtype) * gain, w.dtype)
    p = da.problem(1, H, T, fh, fw, 128, 8, pw, keep_blocks=keep)
    dims = da.da_derive(p)
    O = empty((1, H, dims.n, 128), w.dtype)
    O.fill_(float("nan"))
    idx = torch.empty((1, H, dims.g, dims.k), dtype=torch.int32, device="cuda")
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    x = [to_dev(t, w.dtype) for t in (Q, K, V)]
    da.da_forward(p, *x, O, ws, idx)
    again = torch.empty_like(O)
    da.da_forward(p, *x, again, ws, idx)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(O).all())
    assert torch.equal(O.view(torch.int16), again.view(torch.int16))     # the order of the walk does not depend on the run
    host, host_idx = to_host_f64(O, w.dtype), idx.cpu().numpy()
    for h in sorted({0, H // 3, H - 2, H - 1} & set(range(H))):
        ref = HeadRef(w, Q[0, h], K[0, h], V[0, h], keep_blocks=keep)
        assert np.array_equal(host_idx[0, h], ref.idx)
        emax, emean = output_error(host[0, h], oa.restore(ref.attention(), ref.inv))
        assert emax <= TOL[w.dtype][0] and emean <= TOL[w.dtype][1], (h, emax, emean)
    assert da.da_wait_failures() == 0
