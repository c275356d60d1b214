"""The bf16 attention with two waves per query block, where their division of a list can go wrong: lists of one entry (one
wave gets none), of odd and even length, around the length from which both waves look at the first entry (16), and of
every block; blocks with at most 32 valid slots (half a tile, one wave's worth of queries); frame counts that leave one to
three frames over.  As generated (most tiles dropped) and with Q scaled down (none).  Against the oracle, within the
build target's bounds for bf16 outputs."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, TOL, empty, output_error, say, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keep", [1, 2, 3, 15, 16, 17, 34, 10 ** 6])
@pytest.mark.parametrize("T,fh,fw,pw,gain", [(4, 12, 28, 8, 1.0), (5, 12, 28, 8, 0.03125), (7, 20, 19, 8, 1.0), (3, 20, 40, 16, 1.0),
                                             (6, 12, 40, 16, 0.03125)])
def test_lists_of_every_length(T, fh, fw, pw, gain, keep):
    import torch
    w = W.Workload("pairs", B=1, H=1, d=128, T=T, fh=fh, fw=fw, pw=pw, seed=fh + T)
    say(f"pairs {T}x{fh}x{fw} window 8x{pw} keep {keep} gain {gain}")
    Q, K, V = W.make_qkv(w)
    Q = W.to_storage(W.storage_to_f64(Q, w.dtype) * gain, w.dtype)
    ref = HeadRef(w, Q[0, 0], K[0, 0], V[0, 0], keep_blocks=keep)
    p = da.problem(1, 1, T, fh, fw, 128, 8, pw, keep_blocks=keep)
    dims = da.da_derive(p)
    O = empty((1, 1, dims.n, 128), w.dtype)
    O.fill_(float("nan"))
    idx = torch.empty((1, 1, dims.g, dims.k), dtype=torch.int32, device="cuda")
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    da.da_forward(p, *(to_dev(x, w.dtype) for x in (Q, K, V)), O, ws, idx)
    torch.cuda.synchronize()
    assert np.array_equal(idx[0, 0].cpu().numpy(), ref.idx)
    emax, emean = output_error(to_host_f64(O, w.dtype)[0, 0], oa.restore(ref.attention(), ref.inv))
    assert emax <= TOL[w.dtype][0] and emean <= TOL[w.dtype][1], (emax, emean)
    assert da.da_wait_failures() == 0
