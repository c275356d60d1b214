"""The float32 attention on the matrix instructions, where it can go wrong: both head dimensions, blocks whose upper
half of queries or keys is all pad (at most 32 valid slots), one block in all, one kept block, block counts that do not
divide by eight (the launch deals stretches of blocks to eight XCDs); rows read in the original order (da_forward) and
reordered with V block-transposed (da_sparse_attn), with the log-sum-exp.

Tolerance: float32 products and sums over at most 64 * k <= 1200 keys, scores up to about 46: a score is off by at most
d * 2^-24 * sum|q_c k_c| / sqrt(d) < 1e-5 and an output (|V| < 5) by less than 1e-4, the bound of the build target."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, empty, output_error, say, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,fh,fw,sparsity", [(1, 3, 5, 0.0), (1, 8, 8, 0.0), (3, 12, 9, 0.5), (2, 20, 33, 0.95),
                                              (3, 17, 24, 0.3)])
def test_f32_attention(T, fh, fw, sparsity, d):
    import torch
    w = W.Workload("f32", B=1, H=2, d=d, T=T, fh=fh, fw=fw, sparsity=sparsity, dtype=W.F32, seed=fh)
    say(f"f32 attention {T}x{fh}x{fw} d={d} s={sparsity}")
    Q, K, V = W.make_qkv(w)
    refs = [HeadRef(w, Q[0, h], K[0, h], V[0, h]) for h in range(w.H)]
    p = da.problem_of(w)
    dims = da.da_derive(p)
    x = [to_dev(t, w.dtype) for t in (Q, K, V)]
    O = empty((1, w.H, dims.n, d), w.dtype)
    O.fill_(float("nan"))
    idx = torch.empty((1, w.H, dims.g, dims.k), dtype=torch.int32, device="cuda")
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    da.da_forward(p, *x, O, ws, idx)
    Qp, Kp, Vt, Op = (empty((1, w.H, dims.n_pad, d), w.dtype) for _ in range(4))
    da.da_permute(p, x[0], Qp, da.DA_REORDER_ROWS)
    da.da_permute(p, x[1], Kp, da.DA_REORDER_ROWS)
    da.da_permute(p, x[2], Vt, da.DA_REORDER_VT)
    lse = torch.empty((1, w.H, dims.n_pad), dtype=torch.float32, device="cuda")
    Op.fill_(float("nan"))
    da.da_sparse_attn(p, Qp, Kp, Vt, idx, Op, lse)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(Op).all())                  # pad rows are written, with finite values
    for h, ref in enumerate(refs):
        assert np.array_equal(idx[0, h].cpu().numpy(), ref.idx)
        want, want_lse = ref.attention(want_lse=True)
        real = ref.perm >= 0
        assert output_error(to_host_f64(Op, w.dtype)[0, h][real], want[real])[0] <= 1e-4
        assert np.abs(lse[0, h].cpu().numpy()[real] - want_lse[real]).max() <= 1e-4
        assert output_error(to_host_f64(O, w.dtype)[0, h], oa.restore(want, ref.inv))[0] <= 1e-4


@pytest.mark.parametrize("T,fh,fw,ph,pw,keep", [(3, 40, 48, 8, 8, 64), (3, 40, 48, 8, 8, 65), (3, 40, 48, 8, 8, 90), (2, 9, 34, 4, 16, 5),
                                                (2, 3, 70, 1, 64, 4), (2, 66, 3, 64, 1, 7), (2, 19, 14, 16, 4, 3)])
def test_f32_steps(T, fh, fw, ph, pw, keep):
    """Lists around and beyond the 64 entries that a wave holds at a time, and windows of every shape with 64 tokens (blocks of
    1 to 64 valid slots: steps that hold fewer than 16 keys, quarters that hold none).  Tolerance as above: at most 5760 keys."""
    import torch
    w = W.Workload("f32_steps", B=1, H=1, d=128, T=T, fh=fh, fw=fw, ph=ph, pw=pw, dtype=W.F32, seed=fh + keep)
    say(f"f32 steps {T}x{fh}x{fw} window {ph}x{pw} keep {keep}")
    Q, K, V = W.make_qkv(w)
    ref = HeadRef(w, Q[0, 0], K[0, 0], V[0, 0], keep_blocks=keep)
    p = da.problem(1, 1, T, fh, fw, 128, ph, pw, dtype=da.DA_F32, keep_blocks=keep)
    dims = da.da_derive(p)
    O = empty((1, 1, dims.n, 128), w.dtype)
    O.fill_(float("nan"))
    idx = torch.empty((1, 1, dims.g, dims.k), dtype=torch.int32, device="cuda")
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    da.da_forward(p, *(to_dev(t, w.dtype) for t in (Q, K, V)), O, ws, idx)
    torch.cuda.synchronize()
    assert np.array_equal(idx[0, 0].cpu().numpy(), ref.idx)
    assert output_error(to_host_f64(O, w.dtype)[0, 0], oa.restore(ref.attention(), ref.inv))[0] <= 1e-4
