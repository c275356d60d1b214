"""float32 attention dealt out in halves of a block, in quarters, or both: a head's result does not depend on which (the four waves of
a workgroup share the keys out alike), so a launch of many heads returns the bits that a launch for each head alone does.
Sizes on both sides of the rule's lines, grids that leave blocks of at most 16, 32 and 48 valid slots, k per row and lists of any
length, both layouts of V, with the log-sum-exp; one head also against the oracle."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import HeadRef, output_error, say, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,T,fh,fw,d", [(5, 1, 30, 52, 128), (4, 2, 30, 52, 128), (4, 3, 30, 52, 128), (11, 2, 12, 70, 128),
                                         (5, 1, 30, 52, 64), (10, 2, 18, 50, 64), (4, 3, 30, 52, 64)])
def test_heads_together_and_alone(H, T, fh, fw, d):
    import torch
    say(f"f32 pieces {H} x {T}x{fh}x{fw} d={d}")
    w = W.Workload("f32_pieces", B=1, H=H, d=d, T=T, fh=fh, fw=fw, sparsity=0.8, dtype=W.F32, seed=H)
    Q, K, V = W.make_qkv(w)
    x = [torch.from_numpy(np.ascontiguousarray(t, dtype=np.float32)).cuda() for t in (Q, K, V)]

    def outputs(heads):
        n = len(heads)
        p = da.problem(1, n, T, fh, fw, d, dtype=da.DA_F32, sparsity=0.8)
        dims = da.da_derive(p)
        q, k, v = (t[:, heads].contiguous() for t in x)
        O, O2 = (torch.full_like(q, float("nan")) for _ in range(2))
        idx = torch.empty((1, n, dims.g, dims.k), dtype=torch.int32, device="cuda")
        da.da_forward(p, q, k, v, O, torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda"), idx)
        sizes = da.da_global_sizes(p)
        row_ptr = torch.empty((1, n, dims.g + 1), dtype=torch.int32, device="cuda")
        cols = torch.zeros((1, n, int(sizes.cap)), dtype=torch.int32, device="cuda")
        da.da_forward_global(p, q, k, v, O2, torch.empty(int(sizes.forward_ws), dtype=torch.uint8, device="cuda"), row_ptr, cols)
        Qp, Kp, Vt, Op = (torch.empty((1, n, dims.n_pad, d), dtype=torch.float32, device="cuda") for _ in range(4))
        da.da_permute(p, q, Qp, da.DA_REORDER_ROWS)
        da.da_permute(p, k, Kp, da.DA_REORDER_ROWS)
        da.da_permute(p, v, Vt, da.DA_REORDER_VT)
        lse = torch.empty((1, n, dims.n_pad), dtype=torch.float32, device="cuda")
        da.da_sparse_attn(p, Qp, Kp, Vt, idx, Op, lse)
        torch.cuda.synchronize()
        return [O, idx, O2, row_ptr, Op, lse]

    together = outputs(list(range(H)))
    for h in range(H):
        for a, b in zip(together, outputs([h])):
            assert torch.equal(a[:, h:h + 1], b), h
    ref = HeadRef(w, Q[0, 1], K[0, 1], V[0, 1])
    assert np.array_equal(together[1][0, 1].cpu().numpy(), ref.idx)
    want = oa.restore(ref.attention(), ref.inv)
    assert output_error(to_host_f64(together[0], W.F32)[0, 1], want)[0] <= 1e-4   # (the bound of the other float32 tests: scores up to about 46, at most 1100 keys)
