"""The bf16 attention's own addressing of query and output rows: windows of every shape with 64 and 128 slots, cut at the
frame's edges (blocks of 1 to 128 valid slots), contiguous tensors and the views of a fused projection.  Rows past the last
token of a block are the neighbour's: what da_forward writes is compared everywhere, what lies between is left alone.
Against the oracle, within the build target's bounds for bf16 outputs."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, TOL, empty, output_error, say, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ph,pw,fh,fw", [(8, 8, 17, 21), (64, 1, 66, 3), (1, 64, 3, 70), (16, 4, 19, 14), (4, 16, 9, 34), (2, 32, 5, 33),
                                         (8, 16, 11, 37), (128, 1, 131, 2), (1, 128, 2, 131), (4, 32, 9, 70), (32, 4, 70, 9)])
@pytest.mark.parametrize("T", [1, 5])
def test_rows_of_every_window(T, ph, pw, fh, fw):
    import torch
    H, B = 2, 2
    w = W.Workload("rows", B=B, H=H, d=128, T=T, fh=fh, fw=fw, ph=ph, pw=pw, seed=fh)
    say(f"query rows {T}x{fh}x{fw} window {ph}x{pw}")
    Q, K, V = W.make_qkv(w)
    Q = W.to_storage(W.storage_to_f64(Q, w.dtype) * 0.25, w.dtype)
    p = da.problem(B, H, T, fh, fw, 128, ph, pw, sparsity=0.5)
    dims = da.da_derive(p)
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    idx = torch.empty((B, H, dims.g, dims.k), dtype=torch.int32, device="cuda")
    O = empty((B, H, dims.n, 128), w.dtype)
    O.fill_(float("nan"))
    x = [to_dev(t, w.dtype) for t in (Q, K, V)]
    da.da_forward(p, *x, O, ws, idx)
    # a fused projection's views in, every other row of a wider buffer out
    buf = empty((B, dims.n, 3, H, 128), w.dtype)
    for i in range(3):
        buf[:, :, i] = x[i].permute(0, 2, 1, 3)
    q, k, v = (buf[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    out = empty((B, dims.n, 2, H, 128), w.dtype)
    out.fill_(7.0)
    o = out[:, :, 1].permute(0, 2, 1, 3)
    da.da_forward_ex(p, q, k, v, o, ws, da.layout_of(q), da.layout_of(o), 0, None)
    torch.cuda.synchronize()
    assert torch.equal(o.contiguous().view(torch.int16), O.view(torch.int16))
    assert bool((out[:, :, 0] == 7.0).all())
    got, host_idx = to_host_f64(O, w.dtype), idx.cpu().numpy()
    for b, h in ((0, 0), (B - 1, H - 1)):
        ref = HeadRef(w, Q[b, h], K[b, h], V[b, h], keep_blocks=dims.k)
        assert np.array_equal(host_idx[b, h], ref.idx)
        emax, emean = output_error(got[b, h], oa.restore(ref.attention(), ref.inv))
        assert emax <= TOL[w.dtype][0] and emean <= TOL[w.dtype][1], (b, h, emax, emean)
