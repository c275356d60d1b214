"""Waves that share a list all start from the scores of their own query block, wherever in the unit that is: frames left over put blocks of
several positions into one unit, and a wave that started from another block's scores would carry out most of its tiles.  Keys that only
matter to their own block's queries (random codes, 80 powers of two and more between a block's own scores and the others'), every
block kept, two waves to a list: of the two, the wave that takes the own block carries out that and what it meets before it, at
most one of the other three own blocks of its workgroup, and the other wave nothing."""
import numpy as np
import pytest

from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import empty, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,fh,fw,pw,H", [(3, 30, 52, 8, 8), (1, 32, 64, 8, 24), (7, 24, 40, 8, 6), (2, 16, 80, 16, 12)])
def test_only_the_own_block_is_carried_out(T, fh, fw, pw, H):
    import torch
    say(f"own block {T}x{fh}x{fw} window 8x{pw} heads {H}")
    p = da.problem(1, H, T, fh, fw, 128, 8, pw)
    dims = da.da_derive(p)
    perm = torch.empty(dims.n_pad, dtype=torch.int32, device="cuda")
    valid = torch.empty(dims.g, dtype=torch.int32, device="cuda")
    da.da_build_perm(p, perm, None, valid)
    tokens, valid = perm.cpu().numpy(), valid.cpu().numpy()
    rng = np.random.default_rng(T)
    code = 4.0 * rng.choice([-1.0, 1.0], size=(H, dims.g, 128))          # own score 181, others at most about 90
    gap = np.einsum("hic,hjc->hij", code, code) / np.sqrt(128)
    assert (np.delete(gap.reshape(H, -1), np.arange(dims.g) * (dims.g + 1), axis=1)).max() < 110
    x = np.zeros((1, H, dims.n, 128))
    real = tokens >= 0
    x[0][:, tokens[real]] = code[:, np.nonzero(real)[0] // dims.block]
    V = rng.normal(size=(1, H, dims.n, 128))
    q, v = (to_dev(W.to_storage(a, W.BF16), W.BF16) for a in (x, V))
    Kp = empty((1, H, dims.n_pad, 128), W.BF16)
    Vt, O = torch.empty_like(Kp), empty((1, H, dims.n, 128), W.BF16)
    da.da_permute(p, q, Kp, da.DA_REORDER_ROWS)
    da.da_permute(p, v, Vt, da.DA_REORDER_VOP)
    idx = torch.arange(dims.g, dtype=torch.int32, device="cuda").repeat(H * dims.g, 1).contiguous()
    counts = torch.zeros(2, dtype=torch.int64, device="cuda")
    da.da_sparse_attn_ex(p, q, Kp, Vt, idx, O, None, 1, counts)
    torch.cuda.synchronize()
    seen, kept = (int(c) for c in counts.cpu())
    query_tiles = H * int(np.ceil(valid / 32).sum())
    tiles = int(np.ceil(valid / 64).sum())
    say(f"  tiles gone through {seen}, carried out {kept}: {kept / query_tiles:.3f} per query tile")
    assert seen == query_tiles * tiles
    assert kept <= 2 * query_tiles * (dims.block // 64)
