"""Pooling by small launches whose patch rows are cut (all 64 loads of a block asked for at once, eight bytes per lane): windows
of every shape, blocks of 1 to 128 valid slots (more than 64: a second turn), both data types, mean and maximum, strided
rows, and the launch sizes on both sides of the line to the other kernel.  Bits as the oracle's; da_forward as well, whose
attention reads the reordered K that the bf16 pass writes."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, TOL, empty, output_error, say, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_pool", [False, True])
@pytest.mark.parametrize("dtype,T,fh,fw,ph,pw,H", [(W.BF16, 2, 30, 52, 8, 8, 3), (W.BF16, 2, 13, 41, 8, 16, 2), (W.BF16, 2, 8, 30, 8, 16, 1),
                                                   (W.BF16, 1, 21, 13, 16, 4, 2), (W.BF16, 3, 1, 1, 8, 8, 2), (W.F32, 2, 30, 52, 8, 8, 2),
                                                   (W.F32, 2, 3, 70, 1, 64, 2), (W.F32, 2, 66, 3, 64, 1, 2), (W.BF16, 9, 30, 52, 8, 8, 16),
                                                   (W.BF16, 10, 30, 52, 8, 8, 16)])
def test_pooled_bits(dtype, T, fh, fw, ph, pw, H, max_pool):
    import torch
    w = W.Workload("pool_small", B=1, H=H, d=128, T=T, fh=fh, fw=fw, ph=ph, pw=pw, dtype=dtype, seed=fh + fw)
    say(f"pool small {dtype} {T}x{fh}x{fw} window {ph}x{pw} heads {H} max {max_pool}")
    Q, K, V = W.make_qkv(w)
    p = da.problem(1, H, T, fh, fw, 128, ph, pw, dtype=da.DA_F32 if dtype == W.F32 else da.DA_BF16, keep_blocks=2,
                   pool=da.DA_POOL_MAX if max_pool else da.DA_POOL_AVG)
    dims = da.da_derive(p)
    g = dims.g
    x = [to_dev(t, dtype) for t in (Q, K, V)]
    qp = torch.empty((1, H, g, 128), dtype=torch.float32, device="cuda")
    kp, logits = torch.empty_like(qp), torch.empty((1, H, g, g), dtype=torch.float32, device="cuda")
    da.da_draft_map(p, x[0], x[1], qp, kp, logits, None)
    # da_forward on token-major buffers (rows 3 * H * 128 apart)
    buf = empty((1, dims.n, 3, H, 128), dtype)
    for i in range(3):
        buf[:, :, i] = x[i].permute(0, 2, 1, 3)
    q, k, v = (buf[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    O = empty((1, H, dims.n, 128), dtype)
    idx = torch.empty((1, H, g, dims.k), dtype=torch.int32, device="cuda")
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    da.da_forward_ex(p, q, k, v, O, ws, da.layout_of(q), None, 0, idx)
    torch.cuda.synchronize()
    hq, hk, hi, ho = qp.cpu().numpy(), kp.cpu().numpy(), idx.cpu().numpy(), to_host_f64(O, dtype)
    for h in (0, H - 1):
        ref = HeadRef(w, Q[0, h], K[0, h], V[0, h], keep_blocks=2, max_pool=max_pool)
        assert np.array_equal(hq[0, h].view(np.uint32), ref.q_pool.view(np.uint32)), "pooled Q bits"
        assert np.array_equal(hk[0, h].view(np.uint32), ref.k_pool.view(np.uint32)), "pooled K bits"
        assert np.array_equal(hi[0, h], ref.idx)
        emax, emean = output_error(ho[0, h], oa.restore(ref.attention(), ref.inv))
        assert emax <= TOL[dtype][0] and emean <= TOL[dtype][1], (h, emax, emean)
