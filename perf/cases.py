"""The calls that a video diffusion transformer makes of this library, as cases to time.

A case is one attention layer (or, for `whole_map` and `stages`, the same layer by another of the library's routes) on
the shapes this repository's workloads use: latent grids of 30x52 (480p), 45x80 (720p) and 48x80, 1 to 65 latent
frames, 24 or 40 heads of 128 or the share of them that one of eight GPUs holds, 8x8 or 8x16 pooling windows, 0 to 95 %
of the key blocks dropped, bfloat16 as a rule and float32 where a layer is checked.

Inputs follow the recipe of paper_2505_14708_amd/workloads.py (smooth fields over time, height and width, plus noise),
evaluated on the GPU.  That recipe makes sharply peaked attention; `gain` scales Q, so that gain 1 is that extreme,
1/32 the other (all scores of a row close together: nothing can be skipped), and what normalised queries and keys
give lies between.
"""
from __future__ import annotations

import math

import torch

from paper_2505_14708_amd import binding as da

F32, BF16 = "f32", "bf16"


def _case(name, T, fh, fw, H, sparsity, *, B=1, d=128, ph=8, pw=8, dtype=BF16, gain=1.0, route="forward",
          layout="plain", pool="avg"):
    return {"name": name, "route": route, "layout": layout, "B": B, "H": H, "T": T, "fh": fh, "fw": fw, "d": d, "ph": ph,
            "pw": pw, "dtype": dtype, "sparsity": sparsity, "gain": gain, "pool": pool}


def listed():
    return [
        # the smallest layer: a float32 model of toy size, stepped through a debugger or a unit test; launches count
        _case("f32_toy", 2, 16, 16, 2, 0.5, d=64, dtype=F32),
        # a float32 layer on three 480p frames, the run that a bf16 deployment is checked against
        _case("f32_480p_3_frames", 3, 30, 52, 4, 0.75, dtype=F32, gain=0.25),
        # one 480p frame (an image, or the first frame of a stream), a guided and an unguided sample in one batch, taken
        # from and returned to the fused projection's token-major buffers
        _case("480p_1_frame_fused", 1, 30, 52, 24, 0.5, B=2, gain=0.25, layout="fused"),
        # the 480p clip, all heads on one GPU
        _case("480p", 21, 30, 52, 24, 0.75),
        # the headline layer: 720p, 33 frames, 24 heads, 90 % dropped ...
        _case("720p_33_frames", 33, 45, 80, 24, 0.9),
        # ... and the same layer where attention is not peaked
        _case("720p_33_frames_flat", 33, 45, 80, 24, 0.9, gain=0.03125),
        # one of eight GPUs of a 40-head model: five heads, fused projection
        _case("720p_21_frames_5_heads_fused", 21, 45, 80, 5, 0.75, gain=0.25, layout="fused"),
        # the longest clip, three of 24 heads (one of eight GPUs), activations kept in block order from layer to layer
        _case("720p_65_frames_3_heads_blocks", 65, 45, 80, 3, 0.9, layout="blocks"),
        # 8x16 windows on the grid they divide
        _case("768p_8x16", 33, 48, 80, 24, 0.9, pw=16, gain=0.25),
        # the threshold over a head's whole map instead of k per row
        _case("720p_whole_map", 17, 45, 80, 8, 0.9, gain=0.25, route="whole_map"),
        # a dense layer, as in the first denoising steps
        _case("480p_dense", 21, 30, 52, 3, 0.0, gain=0.25),
        # stage by stage: draft map with its softmax and mask for inspection, reorders, attention with its
        # log-sum-exp, restore
        _case("480p_stages", 9, 30, 52, 8, 0.8, gain=0.25, route="stages"),
    ]


def draw(rng):
    """One more case of the same ranges: frames and heads over their logarithm, any grid between a part of a 480p
    frame and 768p, odd sizes as likely as even ones."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    dtype = F32 if rng.random() < 0.2 else BF16
    route = rng.choices(["forward", "whole_map", "stages"], [6, 1, 1])[0]
    layout = rng.choice(["plain", "fused", "blocks"]) if route == "forward" and dtype == BF16 else "plain"
    c = _case("", log_int(1, 33), rng.randint(12, 48), rng.randint(16, 80), log_int(1, 24),
              rng.choice([0.0, 0.5, 0.6, 0.75, 0.8, 0.9, 0.95]), B=rng.choice([1, 1, 2]),
              d=rng.choice([64, 128]) if dtype == F32 else 128,
              pw=16 if dtype == BF16 and rng.random() < 0.2 else 8, dtype=dtype,
              gain=rng.choice([1.0, 0.25, 0.03125]), route=route, layout=layout,
              pool="max" if rng.random() < 0.15 else "avg")
    # no more than the largest listed case (the flat headline layer), float32 work counted by what its rate makes of
    # it; lists of any length go up to about 7000 blocks
    while _pairs(c) * (64 if dtype == F32 else 1) > 3.0e10 or c["T"] * -(-c["fh"] // 8) * -(-c["fw"] // c["pw"]) > 4000:
        if c["B"] * c["H"] > 1:
            c["B"], c["H"] = 1, max(1, c["H"] // 2)
        else:
            c["T"] = max(1, c["T"] * 3 // 4)
    del c["name"]
    return c


def _problem(c):
    return da.problem(c["B"], c["H"], c["T"], c["fh"], c["fw"], c["d"], c["ph"], c["pw"],
                      dtype=da.DA_F32 if c["dtype"] == F32 else da.DA_BF16, sparsity=c["sparsity"],
                      pool=da.DA_POOL_MAX if c["pool"] == "max" else da.DA_POOL_AVG)


def _pairs(c):
    """Query-key pairs that are kept."""
    dims = da.da_derive(_problem(c))
    n = c["T"] * c["fh"] * c["fw"]
    return c["B"] * c["H"] * float(n) * n * dims.k / dims.g


def _smooth_head(c, gen):
    """Sum of eight random Fourier modes per channel over (t, y, x): [T, fh, fw, d] float32."""
    T, fh, fw, d = c["T"], c["fh"], c["fw"], c["d"]
    f = (torch.rand((d, 8, 3), generator=gen, device="cuda") * 2 - 1) / 16
    phi = torch.rand((d, 8), generator=gen, device="cuda") * (2 * math.pi)
    axis = [2 * math.pi * torch.arange(n, device="cuda", dtype=torch.float32) for n in (T, fh, fw)]
    ty = (phi[:, None, None, :] + axis[0][None, :, None, None] * f[:, None, None, :, 0]
          + axis[1][None, None, :, None] * f[:, None, None, :, 1]).reshape(d, T * fh, 8)
    x = axis[2][None, None, :] * f[:, :, 2, None]                                   # [d, 8, fw]
    field = torch.bmm(torch.cat([ty.cos(), -ty.sin()], 2), torch.cat([x.cos(), x.sin()], 1))   # [d, T*fh, fw]
    return field.permute(1, 2, 0).reshape(T, fh, fw, d)


def _to_blocks(c, dims, x):
    """[B, H, N, d] in token order -> [B, H, n_pad, d] in block order (pad rows zero)."""
    y = torch.zeros((c["B"], c["H"], dims.n_pad, c["d"]), dtype=x.dtype, device=x.device)
    inv = torch.empty(dims.n, dtype=torch.int32, device=x.device)
    da.da_build_perm(_problem(c), None, inv, None)
    y[:, :, inv.long()] = x
    return y


def prepare(case, seed):
    c = case
    p = _problem(c)
    dims = da.da_derive(p)
    B, H, d, n = c["B"], c["H"], c["d"], int(dims.n)
    dt = torch.float32 if c["dtype"] == F32 else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if c["layout"] == "fused":
        buf = torch.empty((B, n, 3, H, d), dtype=dt, device="cuda")
        q, k, v = (buf[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    else:
        q, k, v = (torch.empty((B, H, n, d), dtype=dt, device="cuda") for _ in range(3))
    for b in range(B):
        for h in range(H):
            s = _smooth_head(c, gen).reshape(n, d)
            q[b, h] = ((s + 0.3 * torch.randn((n, d), generator=gen, device="cuda")) * c["gain"]).to(dt)
            k[b, h] = (s + 0.3 * torch.randn((n, d), generator=gen, device="cuda")).to(dt)
            v[b, h] = torch.randn((n, d), generator=gen, device="cuda").to(dt)
    st = {"case": c, "p": p, "dims": dims}
    if c["layout"] == "fused":
        st["O"] = torch.empty((B, n, H, d), dtype=dt, device="cuda").permute(0, 2, 1, 3)
        st["in"], st["out"] = da.layout_of(q), da.layout_of(st["O"])
    elif c["layout"] == "blocks":
        q, k, v = (_to_blocks(c, dims, x) for x in (q, k, v))
        st["O"] = torch.zeros_like(q)
    else:
        st["O"] = torch.empty((B, H, n, d), dtype=dt, device="cuda")
    st["Q"], st["K"], st["V"] = q, k, v
    g = int(dims.g)

    def dev(shape, dtype):
        return torch.empty(shape, dtype=dtype, device="cuda")

    if c["route"] == "whole_map":
        sizes = da.da_global_sizes(p)
        st["ws"] = dev(int(sizes.forward_ws), torch.uint8)
        st["row_ptr"] = dev((B, H, g + 1), torch.int32)
        # (what lies behind a head's last list is not written: start it at a known value)
        st["cols"] = torch.zeros((B, H, int(sizes.cap)), dtype=torch.int32, device="cuda")
    else:
        st["idx"] = dev((B, H, g, int(dims.k)), torch.int32)
    if c["route"] == "forward":
        st["ws"] = dev(da.da_workspace_size(p), torch.uint8)
    if c["route"] == "stages":
        np_ = int(dims.n_pad)
        st["q_pool"], st["k_pool"] = dev((B, H, g, d), torch.float32), dev((B, H, g, d), torch.float32)
        st["logits"], st["draft"] = dev((B, H, g, g), torch.float32), dev((B, H, g, g), torch.float32)
        st["mask"] = dev((B, H, g, g), torch.uint8)
        st["Qp"], st["Kp"], st["Vt"], st["Op"] = (dev((B, H, np_, d), dt) for _ in range(4))
        st["lse"] = dev((B, H, np_), torch.float32)
        st["valid"] = dev(np_, torch.int32)
        da.da_build_perm(p, st["valid"], None, None)
    torch.cuda.synchronize()
    return st


def run(state):
    s = state
    c, p = s["case"], s["p"]
    if c["route"] == "whole_map":
        da.da_forward_global(p, s["Q"], s["K"], s["V"], s["O"], s["ws"], s["row_ptr"], s["cols"])
        return {"O": s["O"], "row_ptr": s["row_ptr"], "cols": s["cols"]}
    if c["route"] == "stages":
        da.da_draft_map(p, s["Q"], s["K"], s["q_pool"], s["k_pool"], s["logits"], s["draft"])
        da.da_select_blocks(p, s["logits"], s["idx"], s["mask"])
        da.da_permute(p, s["Q"], s["Qp"], da.DA_REORDER_ROWS)
        da.da_permute(p, s["K"], s["Kp"], da.DA_REORDER_ROWS)
        da.da_permute(p, s["V"], s["Vt"], da.v_layout(p.dtype))
        da.da_sparse_attn(p, s["Qp"], s["Kp"], s["Vt"], s["idx"], s["Op"], s["lse"])
        da.da_permute(p, s["Op"], s["O"], da.DA_RESTORE)
        # rows of pad slots hold no defined log-sum-exp: a caller masks them out
        lse = s["lse"].masked_fill(s["valid"] < 0, 0.0)
        return {"O": s["O"], "idx": s["idx"], "mask": s["mask"], "draft": s["draft"], "logits": s["logits"],
                "q_pool": s["q_pool"], "k_pool": s["k_pool"], "lse": lse}
    if c["layout"] == "fused":
        da.da_forward_ex(p, s["Q"], s["K"], s["V"], s["O"], s["ws"], s["in"], s["out"], 0, s["idx"])
    elif c["layout"] == "blocks":
        da.da_forward_ex(p, s["Q"], s["K"], s["V"], s["O"], s["ws"], None, None, 1, s["idx"])
    else:
        da.da_forward(p, s["Q"], s["K"], s["V"], s["O"], s["ws"], s["idx"])
    return {"O": s["O"], "idx": s["idx"]}


def work(case):
    """Q, K, V in and O and the lists out, once each; two products over the kept pairs, and the draft logits where
    there is something to rank."""
    c = case
    dims = da.da_derive(_problem(c))
    bh, d, g, k = c["B"] * c["H"], c["d"], int(dims.g), int(dims.k)
    size = 4 if c["dtype"] == F32 else 2
    nbytes = bh * (4.0 * dims.n * d * size + 4.0 * g * k)
    flops = 4.0 * d * _pairs(c)
    if c["route"] == "stages" or k < g:
        flops += 2.0 * bh * g * g * d
    if c["route"] == "stages":
        nbytes += bh * (9.0 * g * g + 8.0 * g * d + 4.0 * dims.n)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Lists, masks and offsets are whole numbers and stay the same.  Against a float64 evaluation over the same lists
    the outputs are off by 2.0e-3 to 2.4e-3 in bf16 (the output's and the probabilities' rounding) and by 1.3e-6 to 6.0e-6 in
    float32 (sums over some hundred to some thousand keys, scores of up to 46); allowed is about four times that."""
    if case["dtype"] == F32:
        return {"rel": 2e-5}
    return {"rel": 1e-2}
