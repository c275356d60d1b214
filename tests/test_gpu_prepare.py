"""Pooling, K's reordering and V's in one launch, or where every block is kept both reorderings and the lists (da_forward, bf16): the bits of lists and output that the same steps one by one
give.  Small and large launches, whole and cut patch rows, blocks of 64 and 128, mean and maximum, contiguous, strided and
block-ordered tensors, the last on both sides of the line where the launches are separate."""
import pytest

from paper_2505_14708_amd import binding as da
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["plain", "fused", "blocks"])
@pytest.mark.parametrize("H,T,fh,fw,pw,pool", [(1, 1, 3, 5, 8, 0), (3, 2, 30, 52, 8, 0), (3, 2, 30, 52, 8, 1), (2, 2, 16, 24, 8, 0), (2, 2, 13, 41, 16, 1),
                                               (36, 1, 30, 52, 8, 0), (37, 1, 30, 52, 8, 0), (16, 10, 30, 52, 8, 0), (64, 1, 16, 64, 8, 1)])
@pytest.mark.parametrize("sparsity", [0.7, 0.0])
def test_same_bits_as_one_by_one(H, T, fh, fw, pw, pool, sparsity, layout):
    import torch
    say(f"prepare {H} x {T}x{fh}x{fw} window 8x{pw} pool {pool} sparsity {sparsity} {layout}")
    p = da.problem(1, H, T, fh, fw, 128, 8, pw, sparsity=sparsity, pool=pool)
    dims = da.da_derive(p)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * T)
    x = [torch.randn((1, H, dims.n, 128), generator=gen, device="cuda").bfloat16() for _ in range(3)]
    # one by one, original order
    qp, kp = (torch.empty((1, H, dims.g, 128), dtype=torch.float32, device="cuda") for _ in range(2))
    logits = torch.empty((1, H, dims.g, dims.g), dtype=torch.float32, device="cuda")
    want_idx, idx = (torch.full((1, H, dims.g, dims.k), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    Kp, Vt = (torch.empty((1, H, dims.n_pad, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    want = torch.empty_like(x[0])
    da.da_draft_map(p, x[0], x[1], qp, kp, logits, None)
    da.da_select_blocks(p, logits, want_idx, None)
    da.da_permute(p, x[1], Kp, da.DA_REORDER_ROWS)
    da.da_permute(p, x[2], Vt, da.DA_REORDER_VOP)
    da.da_sparse_attn_ex(p, x[0], Kp, Vt, want_idx, want, None, 1)
    ws = torch.empty(da.da_workspace_size(p), dtype=torch.uint8, device="cuda")
    if layout == "fused":
        buf = torch.empty((1, dims.n, 3, H, 128), dtype=torch.bfloat16, device="cuda")
        for i in range(3):
            buf[:, :, i] = x[i].permute(0, 2, 1, 3)
        q, k, v = (buf[:, :, i].permute(0, 2, 1, 3) for i in range(3))
        O = torch.empty_like(want)
        da.da_forward_ex(p, q, k, v, O, ws, da.layout_of(q), None, 0, idx)
    elif layout == "blocks":
        q, k, v = (torch.empty_like(Kp) for _ in range(3))
        for src, dst in zip(x, (q, k, v)):
            da.da_permute(p, src, dst, da.DA_REORDER_ROWS)
        Op, O = torch.empty_like(Kp), torch.empty_like(want)
        da.da_forward_ex(p, q, k, v, Op, ws, None, None, 1, idx)
        da.da_permute(p, Op, O, da.DA_RESTORE)
    else:
        O = torch.empty_like(want)
        da.da_forward(p, *x, O, ws, idx)
        if sparsity == 0.0:                                # the whole-map route: the same lists, with offsets
            sizes = da.da_global_sizes(p)
            row_ptr = torch.full((1, H, dims.g + 1), -1, dtype=torch.int32, device="cuda")
            cols = torch.full((1, H, int(sizes.cap)), -1, dtype=torch.int32, device="cuda")
            da.da_forward_global(p, *x, torch.empty_like(want), torch.empty(int(sizes.forward_ws), dtype=torch.uint8, device="cuda"),
                                 row_ptr, cols)
            assert torch.equal(row_ptr[0, -1].cpu(), torch.arange(dims.g + 1, dtype=torch.int32) * dims.g)
            assert torch.equal(cols[:, :, :dims.g * dims.g].reshape(want_idx.shape), want_idx)
    torch.cuda.synchronize()
    assert torch.equal(idx, want_idx)
    assert torch.equal(O.view(torch.int16), want.view(torch.int16))
