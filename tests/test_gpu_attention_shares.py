"""The bf16 attention where a launch does not fill the chip and its units are shared out among two, four or eight workgroups, or
whole but fewer than a round.  Frames that fill groups and frames left over (shares without a group are not launched), a number of patch
positions that does not divide by eight, 128-token blocks whose second half is all pad.  As generated (most tiles dropped) and with Q scaled
down (none).  Every head against the oracle, within the build target's bounds for bf16 outputs."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, TOL, empty, output_error, say, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


# (T, fh, fw, pw, heads, kept blocks): a unit is shared by 2^... workgroups
SHARED = {(1, 30, 52, 8, 24, 5): (1,), (1, 30, 52, 8, 40, 20): (0,), (4, 20, 28, 8, 22, 3): (0,), (2, 20, 40, 16, 30, 4): (0,),
          (5, 20, 40, 8, 6, 17): (2,), (2, 18, 36, 16, 14, 6): (2,), (1, 30, 52, 8, 9, 28): (3,), (3, 13, 57, 8, 4, 40): (3,),
          (3, 18, 36, 16, 3, 19): (3,)}


@pytest.mark.parametrize("gain", [1.0, 0.03125])
@pytest.mark.parametrize("T,fh,fw,pw,H,keep", list(SHARED))
def test_shared_out_workgroups(T, fh, fw, pw, H, keep, gain):
    import torch
    w = W.Workload("shares", B=1, H=H, d=128, T=T, fh=fh, fw=fw, pw=pw, seed=fh + T)
    say(f"shares {T}x{fh}x{fw} window 8x{pw} heads {H} keep {keep} gain {gain}")
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
    # the stages as well: pad rows are written (zeros or finite), with the log-sum-exp
    Qp, Kp, Vt, Op = (empty((1, H, dims.n_pad, 128), w.dtype) for _ in range(4))
    da.da_permute(p, x[0], Qp, da.DA_REORDER_ROWS)
    da.da_permute(p, x[1], Kp, da.DA_REORDER_ROWS)
    da.da_permute(p, x[2], Vt, da.v_layout(p.dtype))
    Op.fill_(float("nan"))
    lse = torch.empty((1, H, dims.n_pad), dtype=torch.float32, device="cuda")
    da.da_sparse_attn(p, Qp, Kp, Vt, idx, Op, lse)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(Op).all())
    host, host_op, host_lse, host_idx = to_host_f64(O, w.dtype), to_host_f64(Op, w.dtype), lse.cpu().numpy(), idx.cpu().numpy()
    for h in range(H):
        ref = HeadRef(w, Q[0, h], K[0, h], V[0, h], keep_blocks=keep)
        assert np.array_equal(host_idx[0, h], ref.idx)
        want, want_lse = ref.attention(want_lse=True)
        real = ref.perm >= 0
        emax, emean = output_error(host[0, h], oa.restore(want, ref.inv))
        assert emax <= TOL[w.dtype][0] and emean <= TOL[w.dtype][1], (h, emax, emean)
        emax, emean = output_error(host_op[0, h][real], want[real])
        assert emax <= TOL[w.dtype][0] and emean <= TOL[w.dtype][1], (h, emax, emean)
        assert np.abs(host_lse[0, h][real] - want_lse[real]).max() <= 2e-2
    assert da.da_wait_failures() == 0
