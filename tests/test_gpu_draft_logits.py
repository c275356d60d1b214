"""Draft logits on the float32 matrix instructions against the oracle's chain of fused multiply-adds, bit for bit: map
sizes around the 64-wide tile and its 32-wide quarters (rows that are and are not a multiple of four columns), channel
counts around the 32-channel stage and the eight and four channels it is read in, and operands of every magnitude
(subnormal products, sums that overflow)."""
import numpy as np
import pytest

from oracle import draft_attention as oa
from paper_2505_14708_amd import binding as da
from paper_2505_14708_amd import workloads as W
from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", ["ordinary", "spread", "subnormal", "huge"])
@pytest.mark.parametrize("g,d", [(1, 4), (31, 12), (32, 28), (33, 32), (63, 36), (64, 40), (65, 44), (130, 64), (132, 100), (257, 128)])
def test_draft_logits_bit_exact(g, d, scale):
    import torch
    rng = np.random.default_rng([g, d])
    say(f"draft logits g={g} d={d} {scale}")
    Q, K = rng.normal(size=(2, 1, 2, g, d))
    if scale == "spread":
        Q, K = Q * 2.0 ** rng.integers(-30, 30, Q.shape), K * 2.0 ** rng.integers(-30, 30, K.shape)
    elif scale == "subnormal":
        Q, K = Q * 1e-22, K * 1e-18
    elif scale == "huge":
        Q, K = Q * 1e18, K * 1e20
    Q, K = Q.astype(np.float32), K.astype(np.float32)
    p = da.problem(1, 2, 1, 1, g, d, 1, 1, dtype=da.DA_F32)      # 1x1 windows: the pooled tensors are Q and K themselves
    qp, kp = (torch.empty((1, 2, g, d), dtype=torch.float32, device="cuda") for _ in range(2))
    logits = torch.full((1, 2, g, g), 7.0, dtype=torch.float32, device="cuda")
    da.da_draft_map(p, to_dev(Q, W.F32), to_dev(K, W.F32), qp, kp, logits, None)
    torch.cuda.synchronize()
    with np.errstate(over="ignore", invalid="ignore"):
        for h in range(2):
            got, want = logits[0, h].cpu().numpy(), oa.draft_logits_canonical_f32(qp[0, h].cpu().numpy(), kp[0, h].cpu().numpy())
            assert np.array_equal(np.isnan(got), np.isnan(want))
            assert np.array_equal(got.view(np.uint32)[~np.isnan(want)], want.view(np.uint32)[~np.isnan(want)])
