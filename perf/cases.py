"""The work that users of this library have it do, as timed cases: shifted-window attention forward
and backward, the rotary embedding, a rank's share of the windows, the projections and their
gradients, the element-wise operations, and whole transformer layers, from launch-bound grids of
one megabyte to the 0.25-degree grid.

listed() are the fixed cases, draw() gives more of the same ranges; prepare() makes what a program
holds before the call, run() is one pass through the public entry points, work() the bytes and
operations it cannot do without, tolerance() how far another correct implementation may differ,
exact() the values in 64 bits.
"""
import ctypes
import math

import torch

from paper_2509_13523_amd import binding as B
from paper_2509_13523_amd import synth

MASKS = {"none": B.AERIS_MASK_NONE, "lat": B.AERIS_MASK_LAT, "swin": B.AERIS_MASK_SWIN}
EPS, ROPE_BASE = 1e-6, 100.0
GRID_025 = dict(B=1, H=720, W=1440)          # the 0.25-degree grid, poles removed


def _attn(kind, B, H, W, heads, d, wh, ww, sh, sw, mask="swin", out="bf16", data="normal", **more):
    return dict(kind=kind, B=B, H=H, W=W, heads=heads, d=d, wh=wh, ww=ww, sh=sh, sw=sw, mask=mask,
                out=out, data=data, **more)


def listed():
    cases = [
        # a tiny test grid, one forward call: nothing but latency (launches, host path)
        ("attn_fwd_small", _attn("attn_fwd", 1, 64, 128, 4, 32, 8, 8, 4, 4)),
        # a training step of one attention layer on a 1-degree-class grid with small windows:
        # bound by memory traffic, not by matrix products
        ("attn_train_1deg", _attn("attn_train", 1, 180, 360, 8, 64, 12, 12, 6, 6)),
        # odd windows, odd shift, five heads, fp32 results, seam on one axis only: what a user on
        # a grid of another resolution meets (nothing is a multiple of a tile)
        ("attn_train_ragged_f32", _attn("attn_train", 2, 115, 184, 5, 64, 23, 23, 11, 7, mask="lat",
                                        out="f32")),
        # inference on the 0.25-degree grid, 60 x 60 windows, head_dim 64
        ("attn_fwd_60x60_d64", _attn("attn_fwd", heads=16, d=64, wh=60, ww=60, sh=30, sw=30, **GRID_025)),
        # the 6-hourly model's windows, head_dim 128: ragged tiles on both sides
        ("attn_train_30x30", _attn("attn_train", heads=16, d=128, wh=30, ww=30, sh=15, sw=15, **GRID_025)),
        # the headline layer: 60 x 60 windows, head_dim 128, one member of the ensemble batch
        # (smooth fields blended with noise: peaked softmax rows)
        ("attn_train_60x60", _attn("attn_train", heads=16, d=128, wh=60, ww=60, sh=30, sw=30,
                                   data="blend", **GRID_025)),
        # one of eight window-parallel ranks: every eighth window, rotary embedding, the rotated
        # operands handed from the forward to the backward call
        ("rope_share_train", _attn("rope_share", heads=16, d=128, wh=60, ww=60, sh=30, sw=30,
                                   every=8, first=3, **GRID_025)),
        # a small model's whole transformer layer, forward and backward: about thirty short launches
        ("layer_train_small", dict(kind="layer", B=2, H=24, W=36, heads=2, d=64, hidden=512, wh=12,
                                   ww=12, sh=6, sw=6, mask="swin")),
        # a latitude band of the 0.25-degree grid (2 x 24 windows) through a whole layer at the
        # full model width: projections, rotary attention on packed QKV, element-wise kernels
        ("layer_train_band", dict(kind="layer", B=1, H=120, W=1440, heads=16, d=128, hidden=5504,
                                  wh=60, ww=60, sh=30, sw=30, mask="swin")),
        # the projections of a layer at inference, a mid-sized model on two coarse samples: fused
        # QKV, output projection, gated up-projection, down-projection; ragged token tiles
        ("proj_fwd", dict(kind="proj_fwd", samples=2, rows=16200, C=1024, hidden=2752)),
        # gradients of a QKV projection with rows that are no multiple of anything
        ("proj_bwd_ragged", dict(kind="proj_bwd", rows=20011, C=768, F=2304)),
        # the element-wise operations of a layer, forward and backward, on the whole 0.25-degree
        # grid at the full width: every one of them bound by memory traffic
        ("layer_ops", dict(kind="layer_ops", samples=1, rows=720 * 1440, C=2048)),
    ]
    return [dict(c, name=name) for name, c in cases]


# ------------------------------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_window(rng, most_tokens):
    """Window sides from 4 to 64 (both odd and even), at most most_tokens tokens, and a shift."""
    while True:
        wh = int(round(_log(rng, 4, 64)))
        ww = wh if rng.random() < 0.7 else int(round(_log(rng, 4, 64)))
        if wh * ww <= most_tokens:
            break
    shifted = rng.random() < 0.7
    sh = rng.choice([wh // 2, rng.randrange(wh)]) if shifted else 0
    sw = rng.choice([ww // 2, rng.randrange(ww)]) if shifted else 0
    return wh, ww, sh, sw


def _draw_grid(rng, tokens, wh, ww):
    """A grid of about `tokens` tokens that the window divides, wider than high."""
    n = max(1, int(round(tokens / (wh * ww))))
    ny = max(1, min(n, int(round(math.sqrt(n / 2) * rng.uniform(0.7, 1.4)))))
    return ny * wh, max(1, n // ny) * ww


def draw(rng):
    kind = rng.choice(["attn_fwd", "attn_fwd", "attn_train", "attn_train", "attn_train", "rope_share",
                       "layer", "proj_fwd", "proj_bwd", "layer_ops"])
    mask = rng.choice(["none", "lat", "swin", "swin"])
    if kind in ("attn_fwd", "attn_train", "rope_share"):
        wh, ww, sh, sw = _draw_window(rng, 3600)
        d, heads = rng.choice([32, 64, 128]), rng.randint(1, 16)
        H, W = _draw_grid(rng, _log(rng, 8e3, 1e6), wh, ww)
        if kind == "rope_share":
            windows = (H // wh) * (W // ww)
            every = rng.randint(1, min(8, windows))
            return _attn(kind, 1, H, W, heads, d, wh, ww, sh, sw, mask, every=every,
                         first=rng.randrange(every))
        out = rng.choice(["bf16", "bf16", "f32"])
        nb = rng.randint(1, 3) if H * W < 250000 else 1
        return _attn(kind, nb, H, W, heads, d, wh, ww, sh, sw, mask, out,
                     data=rng.choice(["normal", "blend"]))
    if kind == "layer":
        wh, ww, sh, sw = _draw_window(rng, 3600)
        d = rng.choice([32, 64, 128])
        heads = max(1, min(16, int(_log(rng, 2, 17))))
        heads = max(heads, 64 // d) // max(1, 64 // d) * max(1, 64 // d)   # channels: multiple of 64
        C = heads * d
        hidden = 64 * max(1, int(round(C * 2.7 / 64)))
        H, W = _draw_grid(rng, _log(rng, 1e3, 1.7e5), wh, ww)
        nb = rng.randint(1, 2) if H * W < 80000 else 1
        return dict(kind=kind, B=nb, H=H, W=W, heads=heads, d=d, hidden=hidden, wh=wh, ww=ww, sh=sh,
                    sw=sw, mask=mask)
    rows, C = int(_log(rng, 500, 2e5)), 64 * int(_log(rng, 2, 33))
    if kind == "proj_fwd":
        samples = rng.randint(1, 4)
        return dict(kind=kind, samples=samples, rows=max(1, rows // samples), C=C,
                    hidden=64 * max(1, int(round(C * 2.7 / 64))))
    if kind == "proj_bwd":
        return dict(kind=kind, rows=rows, C=C, F=C * rng.choice([1, 3, 5]))
    samples = rng.randint(1, 4)
    return dict(kind=kind, samples=samples, rows=max(1, rows * 4 // samples),
                C=8 * int(_log(rng, 8, 320)))


# ------------------------------------------------------------------------------------- preparation
def _out_dtype(case):
    return B.AERIS_DT_F32 if case.get("out") == "f32" else B.AERIS_DT_BF16


class _Inputs:
    """Device tensors drawn from one generator."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def bf16(self, *shape, scale=1.0):
        t = torch.randn(*shape, device="cuda", dtype=torch.bfloat16, generator=self.gen)
        return t.mul_(scale) if scale != 1.0 else t

    def f32(self, *shape, scale=1.0, mean=0.0):
        return mean + scale * torch.randn(*shape, device="cuda", generator=self.gen)


def _share(case):
    n = (case["H"] // case["wh"]) * (case["W"] // case["ww"])
    return [w for w in range(n) if w % case["every"] == case["first"]]


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    inp = _Inputs(seed)
    if kind in ("attn_fwd", "attn_train", "rope_share"):
        shape = (case["B"], case["H"], case["W"], case["heads"], case["d"])
        s["t"] = synth.make_inputs_device(case["data"], 1000 * (seed % 1000003), shape,
                                          3 if kind == "attn_fwd" else 4)
        s["win"], s["shift"], s["mask"] = (case["wh"], case["ww"]), (case["sh"], case["sw"]), MASKS[case["mask"]]
        if kind == "rope_share":
            s["windows"] = torch.tensor(_share(case), dtype=torch.int32, device="cuda")
            # a rank's full-grid buffers; the calls write the share's windows only
            s["o"], s["dq"], s["dk"], s["dv"] = [torch.zeros_like(s["t"][0]) for _ in range(4)]
            s["lse"] = torch.zeros(shape[0], shape[3], shape[1], shape[2], device="cuda")
            p = B.make_params(shape, s["win"], s["shift"], s["mask"])
            s["saved"] = torch.empty(B.aeris_winattn_rope_fwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
            s["ws"] = torch.empty(B.aeris_winattn_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    elif kind == "layer":
        nb, H, W, nh, d, hidden = [case[k] for k in ("B", "H", "W", "heads", "d", "hidden")]
        C, rps = nh * d, H * W
        N = nb * rps
        s["x"], s["dout"] = inp.bf16(N, C), inp.bf16(N, C)
        s["wqkv"], s["wo"] = inp.bf16(3 * C, C, scale=C ** -0.5), inp.bf16(C, C, scale=C ** -0.5)
        s["wup"], s["wdown"] = inp.bf16(2 * hidden, C, scale=C ** -0.5), inp.bf16(C, hidden, scale=hidden ** -0.5)
        for i in "12":
            s["w" + i] = inp.f32(C, scale=0.1, mean=1.0)
            s["g" + i], s["b" + i], s["a" + i] = (inp.f32(nb, C, scale=0.3), inp.f32(nb, C, scale=0.5),
                                                  inp.f32(nb, C, scale=0.8))
        s["p"] = B.make_params((nb, H, W, nh, d), (case["wh"], case["ww"]), (case["sh"], case["sw"]),
                               MASKS[case["mask"]], qkv_strides=(3 * C, d))
        s["rp"] = B.aeris_rope_params(ROPE_BASE, B.AERIS_ROPE_POS_WINDOW)
        u8 = lambda n: torch.empty(max(int(n), 16), dtype=torch.uint8, device="cuda")
        s["ws_proj"] = u8(max(B.aeris_norm_linear_workspace_bytes(N, rps, C, 2 * hidden),
                              B.aeris_norm_linear_workspace_bytes(N, rps, C, 3 * C)))
        s["ws_attn_f"] = u8(B.aeris_winattn_rope_fwd_workspace_bytes(s["p"]))
        s["ws_attn_b"] = u8(B.aeris_winattn_bwd_workspace_bytes(s["p"]))
        s["ws_lin"] = u8(max(B.aeris_linear_bwd_workspace_bytes(N, C, 2 * hidden),
                             B.aeris_linear_bwd_workspace_bytes(N, hidden, C),
                             B.aeris_linear_bwd_workspace_bytes(N, C, 3 * C),
                             B.aeris_linear_bwd_workspace_bytes(N, C, C)))
        s["ws_el"] = u8(max(B.aeris_rmsnorm_adaln_bwd_workspace_bytes(N, rps, C),
                            B.aeris_gate_residual_bwd_workspace_bytes(N, rps, C)))
    elif kind == "proj_fwd":
        C, hidden, N = case["C"], case["hidden"], case["samples"] * case["rows"]
        s["x"], s["g"] = inp.bf16(N, C), inp.bf16(N, hidden, scale=0.5)
        s["wqkv"], s["wo"] = inp.bf16(3 * C, C, scale=C ** -0.5), inp.bf16(C, C, scale=C ** -0.5)
        s["wup"], s["wdown"] = inp.bf16(2 * hidden, C, scale=C ** -0.5), inp.bf16(C, hidden, scale=hidden ** -0.5)
        s["w"] = inp.f32(C, scale=0.1, mean=1.0)
        s["gamma"], s["beta"] = inp.f32(case["samples"], C, scale=0.3), inp.f32(case["samples"], C, scale=0.5)
        s["ws"] = torch.empty(max(B.aeris_norm_linear_workspace_bytes(N, case["rows"], C, 2 * hidden),
                                  B.aeris_norm_linear_workspace_bytes(N, case["rows"], C, 3 * C)),
                              dtype=torch.uint8, device="cuda")
    elif kind == "proj_bwd":
        N, C, F = case["rows"], case["C"], case["F"]
        s["x"], s["dy"], s["w"] = inp.bf16(N, C), inp.bf16(N, F), inp.bf16(F, C, scale=C ** -0.5)
        s["ws"] = torch.empty(max(16, B.aeris_linear_bwd_workspace_bytes(N, C, F)), dtype=torch.uint8, device="cuda")
    else:
        C, nb, rps = case["C"], case["samples"], case["rows"]
        N = nb * rps
        s["x"], s["y"], s["d"] = inp.bf16(N, C), inp.bf16(N, C), inp.bf16(N, C)
        s["uv"], s["dg"] = inp.bf16(N, 2 * C), inp.bf16(N, C)
        s["w"] = inp.f32(C, scale=0.1, mean=1.0)
        s["gamma"], s["beta"], s["alpha"] = (inp.f32(nb, C, scale=0.3), inp.f32(nb, C, scale=0.5),
                                             inp.f32(nb, C, scale=0.8))
        s["ws"] = torch.empty(max(16, B.aeris_rmsnorm_adaln_bwd_workspace_bytes(N, rps, C),
                                  B.aeris_gate_residual_bwd_workspace_bytes(N, rps, C)),
                              dtype=torch.uint8, device="cuda")
    return s


# ------------------------------------------------------------------------------------- one pass
def _packed_attention(s, call, qkv, *rest):
    """A rotary attention call on the packed [tokens, 3C] projection, through the C entry points
    (the stride fields of the parameter block describe the packing)."""
    C = qkv.shape[1] // 3
    part = lambda t, i: t.data_ptr() + i * C * 2
    rc = call(ctypes.byref(s["p"]), ctypes.byref(s["rp"]), part(qkv, 0), part(qkv, 1), part(qkv, 2),
              *rest, torch.cuda.current_stream().cuda_stream)
    if rc != 0:
        raise B.AerisError(rc, "packed attention")


def _layer(s):
    """Adaptive RMSNorm -> QKV projection -> rotary shifted-window attention -> output projection
    -> gated residual; adaptive RMSNorm -> SwiGLU -> down projection -> gated residual; and the
    backward pass of all of it.  Returns the output and every gradient."""
    x, dout = s["x"], s["dout"]
    rps = s["case"]["H"] * s["case"]["W"]
    N, C = x.shape
    lib, p = B.load(), s["p"]
    a = torch.empty_like(x)
    lse = torch.empty(p.B, p.heads, p.H_lat, p.W_lon, device=x.device)
    qkv = B.aeris_norm_linear_fwd(x, s["w1"], s["g1"], s["b1"], EPS, s["wqkv"], rps, workspace=s["ws_proj"])
    _packed_attention(s, lib.aeris_winattn_rope_fwd, qkv, a.data_ptr(), lse.data_ptr(),
                      s["ws_attn_f"].data_ptr(), s["ws_attn_f"].numel())
    y = B.aeris_linear_fwd(a, s["wo"])
    x1 = B.aeris_gate_residual_fwd(x, y, s["a1"], rps)
    g, uv = B.aeris_norm_linear_swiglu_fwd(x1, s["w2"], s["g2"], s["b2"], EPS, s["wup"], rps,
                                           workspace=s["ws_proj"])
    y2 = B.aeris_linear_fwd(g, s["wdown"])
    out = B.aeris_gate_residual_fwd(x1, y2, s["a2"], rps)

    dy2, da2 = B.aeris_gate_residual_bwd(y2, s["a2"], dout, rps, workspace=s["ws_el"])
    dg, dwdown = B.aeris_linear_bwd(g, s["wdown"], dy2, workspace=s["ws_lin"])
    duv = B.aeris_swiglu_bwd(uv, dg)
    h2, r2 = B.aeris_rmsnorm_adaln_fwd(x1, s["w2"], s["g2"], s["b2"], EPS, rps)
    dh2, dwup = B.aeris_linear_bwd(h2, s["wup"], duv, workspace=s["ws_lin"])
    dx1, dw2, dg2, db2 = B.aeris_rmsnorm_adaln_bwd(x1, s["w2"], s["g2"], r2, dh2, rps,
                                                   workspace=s["ws_el"], dres=dout)
    dy, da1 = B.aeris_gate_residual_bwd(y, s["a1"], dx1, rps, workspace=s["ws_el"])
    da, dwo = B.aeris_linear_bwd(a, s["wo"], dy, workspace=s["ws_lin"])
    dqkv = torch.empty_like(qkv)
    part = lambda t, i: t.data_ptr() + i * C * 2
    _packed_attention(s, lib.aeris_winattn_rope_bwd, qkv, a.data_ptr(), lse.data_ptr(), da.data_ptr(),
                      part(dqkv, 0), part(dqkv, 1), part(dqkv, 2), s["ws_attn_f"].data_ptr(),
                      s["ws_attn_b"].data_ptr(), s["ws_attn_b"].numel())
    h1, r1 = B.aeris_rmsnorm_adaln_fwd(x, s["w1"], s["g1"], s["b1"], EPS, rps)
    dh1, dwqkv = B.aeris_linear_bwd(h1, s["wqkv"], dqkv, workspace=s["ws_lin"])
    dx, dw1, dg1, db1 = B.aeris_rmsnorm_adaln_bwd(x, s["w1"], s["g1"], r1, dh1, rps,
                                                  workspace=s["ws_el"], dres=dx1)
    return dict(out=out, dx=dx, dwqkv=dwqkv, dwo=dwo, dwup=dwup, dwdown=dwdown, dw1=dw1, dg1=dg1,
                db1=db1, da1=da1, dw2=dw2, dg2=dg2, db2=db2, da2=da2)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "attn_fwd":
        q, k, v = s["t"]
        return B.aeris_winattn_fwd(q, k, v, s["win"], s["shift"], s["mask"], out_dtype=_out_dtype(case))
    if kind == "attn_train":
        q, k, v, do = s["t"]
        o, lse = B.aeris_winattn_fwd(q, k, v, s["win"], s["shift"], s["mask"], out_dtype=_out_dtype(case))
        dq, dk, dv = B.aeris_winattn_bwd(q, k, v, o, lse, do, s["win"], s["shift"], s["mask"],
                                         out_dtype=_out_dtype(case))
        return dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)
    if kind == "rope_share":
        q, k, v, do = s["t"]
        rope = (ROPE_BASE, B.AERIS_ROPE_POS_WINDOW)
        o, lse = B.aeris_winattn_rope_fwd_windows(q, k, v, s["win"], s["shift"], *rope, s["windows"],
                                                  s["o"], s["lse"], s["mask"], workspace=s["saved"])
        dq, dk, dv = B.aeris_winattn_rope_bwd_windows(q, k, v, o, lse, do, s["win"], s["shift"], *rope,
                                                      s["windows"], s["dq"], s["dk"], s["dv"], s["mask"],
                                                      workspace=s["ws"], saved=s["saved"])
        return dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)
    if kind == "layer":
        return _layer(s)
    if kind == "proj_fwd":
        rows = case["rows"]
        qkv = B.aeris_norm_linear_fwd(s["x"], s["w"], s["gamma"], s["beta"], EPS, s["wqkv"], rows,
                                      workspace=s["ws"])
        y = B.aeris_linear_fwd(s["x"], s["wo"])
        g, _ = B.aeris_norm_linear_swiglu_fwd(s["x"], s["w"], s["gamma"], s["beta"], EPS, s["wup"], rows,
                                              want_uv=False, workspace=s["ws"])
        y2 = B.aeris_linear_fwd(s["g"], s["wdown"])
        return dict(qkv=qkv, y=y, g=g, y2=y2)
    if kind == "proj_bwd":
        dx, dw = B.aeris_linear_bwd(s["x"], s["w"], s["dy"], workspace=s["ws"])
        return dict(dx=dx, dw=dw)
    rows = case["rows"]
    h, r = B.aeris_rmsnorm_adaln_fwd(s["x"], s["w"], s["gamma"], s["beta"], EPS, rows)
    dx, dw, dgamma, dbeta = B.aeris_rmsnorm_adaln_bwd(s["x"], s["w"], s["gamma"], r, s["d"], rows,
                                                      workspace=s["ws"], dres=s["y"])
    out = B.aeris_gate_residual_fwd(s["x"], s["y"], s["alpha"], rows)
    dy, dalpha = B.aeris_gate_residual_bwd(s["y"], s["alpha"], s["d"], rows, workspace=s["ws"])
    g = B.aeris_swiglu_fwd(s["uv"])
    duv = B.aeris_swiglu_bwd(s["uv"], s["dg"])
    return dict(h=h, r=r, dx=dx, dw=dw, dgamma=dgamma, dbeta=dbeta, out=out, dy=dy, dalpha=dalpha, g=g, duv=duv)


# ------------------------------------------------------------------------------------- 64-bit values
def _partition(case, windows=None):
    """(grid index, region) of every window's tokens, [windows, tokens]: the cyclic shift, and the
    seam rules of the mask."""
    H, W, wh, ww, sh, sw = [case[k] for k in ("H", "W", "wh", "ww", "sh", "sw")]
    n = torch.arange((H // wh) * (W // ww), device="cuda") if windows is None else torch.tensor(windows, device="cuda")
    t = torch.arange(wh * ww, device="cuda")
    yh = (n // (W // ww) * wh)[:, None] + (t // ww)[None]
    xh = (n % (W // ww) * ww)[:, None] + (t % ww)[None]
    region = torch.zeros_like(yh)
    if case["mask"] != "none":
        region += 2 * (yh >= H - sh) * (sh > 0)
    if case["mask"] == "swin":
        region += (xh >= W - sw) * (sw > 0)
    last = ((yh >= H - wh).int() * 2 + (xh >= W - ww).int()) * 4      # other windows never meet a seam
    return (yh + sh) % H * W + (xh + sw) % W, region + last


def _attention64(case, q, k, v, do=None, windows=None):
    """Attention inside the windows and, with dO, its gradients; q .. dO are [B, H, W, heads, d]."""
    idx, region = _partition(case, windows)
    nb, H, W, nh, d = q.shape
    n, T = idx.shape
    flat = lambda t: t.reshape(nb, H * W, nh, d)
    new = lambda: torch.zeros(nb, H * W, nh, d, dtype=torch.float64, device="cuda")
    o, lse = new(), torch.zeros(nb, nh, H * W, dtype=torch.float64, device="cuda")
    grads = [new() for _ in range(3)] if do is not None else []
    step = max(1, int(1.7e9 / (nh * T * T * 8)))
    for b in range(nb):
        for i in range(0, n, step):
            at, reg = idx[i:i + step], region[i:i + step]
            rows = lambda t: flat(t)[b][at].permute(0, 2, 1, 3).to(torch.float64, memory_format=torch.contiguous_format)
            turned = lambda t: t.transpose(-1, -2).contiguous()
            Q, K, V = rows(q), rows(k), rows(v)
            P = Q @ turned(K)
            P.mul_(d ** -0.5)
            if bool((reg != reg[:, :1]).any()):
                P.masked_fill_((reg[:, :, None] != reg[:, None, :])[:, None], -math.inf)
            L = torch.logsumexp(P, -1)
            P.sub_(L[..., None]).exp_()
            O = P @ V
            o[b][at] = O.permute(0, 2, 1, 3)
            lse[b][:, at] = L.permute(1, 0, 2)
            if do is None:
                continue
            dO = rows(do)
            grads[2][b][at] = (turned(P) @ dO).permute(0, 2, 1, 3)
            dS = dO @ turned(V)
            dS.sub_((dO * O).sum(-1, keepdim=True)).mul_(P).mul_(d ** -0.5)
            grads[0][b][at] = (dS @ K).permute(0, 2, 1, 3)
            grads[1][b][at] = (turned(dS) @ Q).permute(0, 2, 1, 3)
    return (o.view(q.shape), lse.view(nb, nh, H, W)) + tuple(g.view(q.shape) for g in grads)


def _rotated64(case, t, back=False):
    """The rotary embedding with positions inside the window: even channel pairs turn with the
    longitude, odd ones with the latitude."""
    H, W, d = case["H"], case["W"], case["d"]
    theta = ROPE_BASE ** (-torch.arange(d // 4, dtype=torch.float64, device="cuda") / (d // 4))
    y = (torch.arange(H, device="cuda") - case["sh"]) % H % case["wh"]
    x = (torch.arange(W, device="cuda") - case["sw"]) % W % case["ww"]
    phi = torch.stack([(x[:, None] * theta)[None].expand(H, -1, -1),
                       (y[:, None] * theta)[:, None].expand(-1, W, -1)], -1).reshape(H, W, 1, d // 2)
    c, s = phi.cos(), -phi.sin() if back else phi.sin()
    a, b = t[..., 0::2].double(), t[..., 1::2].double()
    return torch.stack([a * c - b * s, a * s + b * c], -1).reshape(t.shape)


class _RotaryAttention64(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, k, v, case):
        ctx.case = case
        ctx.save_for_backward(q, k, v)
        return _attention64(case, _rotated64(case, q), _rotated64(case, k), v)[0]

    @staticmethod
    def backward(ctx, do):
        q, k, v = ctx.saved_tensors
        case = ctx.case
        _, _, dq, dk, dv = _attention64(case, _rotated64(case, q), _rotated64(case, k), v, do)
        return _rotated64(case, dq, True), _rotated64(case, dk, True), dv, None


def _norm64(x, w, gamma, beta, rows):
    n = x * torch.rsqrt((x * x).mean(1, keepdim=True) + EPS)
    per_row = lambda t: t.repeat_interleave(rows, 0)
    return n * w * (1 + per_row(gamma)) + per_row(beta)


def _silu_gate64(uv):
    u, v = uv.chunk(2, 1)
    return u * torch.sigmoid(u) * v


def exact(case, seed):
    """What run() returns, in 64 bits; None where that would take long or not fit."""
    kind, amount = case["kind"], work(case)
    if amount["flops"] > 1.2e14 or (kind == "layer_ops" and amount["bytes"] > 1e10):
        return None
    s = prepare(case, seed)
    if kind == "attn_fwd":
        return _attention64(case, *s["t"])
    if kind == "attn_train":
        return dict(zip(("o", "lse", "dq", "dk", "dv"), _attention64(case, *s["t"])))
    if kind == "rope_share":
        q, k, v, do = s["t"]
        o, lse, dq, dk, dv = _attention64(case, _rotated64(case, q), _rotated64(case, k), v, do, _share(case))
        return dict(o=o, lse=lse, dq=_rotated64(case, dq, True), dk=_rotated64(case, dk, True), dv=dv)
    p = {n: t.double() for n, t in s.items() if torch.is_tensor(t) and t.dtype != torch.uint8}
    s.clear()
    if kind == "proj_fwd":
        h = _norm64(p["x"], p["w"], p["gamma"], p["beta"], case["rows"])
        return dict(qkv=h @ p["wqkv"].t(), y=p["x"] @ p["wo"].t(), g=_silu_gate64(h @ p["wup"].t()),
                    y2=p["g"] @ p["wdown"].t())
    if kind == "proj_bwd":
        return dict(dx=p["dy"] @ p["w"], dw=p["dy"].t() @ p["x"])
    if kind == "layer_ops":
        rows, x = case["rows"], p["x"].requires_grad_()
        par = [p[n].requires_grad_() for n in ("w", "gamma", "beta")]
        h = _norm64(x, *par, rows)
        dx, dw, dgamma, dbeta = torch.autograd.grad(h, [x] + par, p["d"])
        y, alpha, uv = [p[n].requires_grad_() for n in ("y", "alpha", "uv")]
        out = x + alpha.repeat_interleave(rows, 0) * y
        dy, dalpha = torch.autograd.grad(out, [y, alpha], p["d"])
        g = _silu_gate64(uv)
        r = torch.rsqrt((x * x).mean(1) + EPS)
        return {n: t.detach() for n, t in dict(
            h=h, r=r, dx=dx + y, dw=dw, dgamma=dgamma, dbeta=dbeta, out=out, dy=dy, dalpha=dalpha, g=g,
            duv=torch.autograd.grad(g, uv, p["dg"])[0]).items()}
    rows, C = case["H"] * case["W"], case["heads"] * case["d"]
    for n, t in p.items():
        t.requires_grad_(n != "dout")
    grid = (case["B"], case["H"], case["W"], case["heads"], case["d"])
    per_row = lambda t: t.repeat_interleave(rows, 0)
    qkv = _norm64(p["x"], p["w1"], p["g1"], p["b1"], rows) @ p["wqkv"].t()
    a = _RotaryAttention64.apply(*[t.reshape(grid) for t in qkv.chunk(3, 1)], case)
    x1 = p["x"] + per_row(p["a1"]) * (a.reshape(-1, C) @ p["wo"].t())
    g = _silu_gate64(_norm64(x1, p["w2"], p["g2"], p["b2"], rows) @ p["wup"].t())
    out = x1 + per_row(p["a2"]) * (g @ p["wdown"].t())
    names = ("x", "wqkv", "wo", "wup", "wdown", "w1", "g1", "b1", "a1", "w2", "g2", "b2", "a2")
    return dict([("out", out.detach())] + [("d" + n, t) for n, t in zip(
        names, torch.autograd.grad(out, [p[n] for n in names], p["dout"]))])


# ------------------------------------------------------------------------------------- accounting
def _visible_pairs(case, windows=None):
    """(query, key) pairs inside a region, per batch member and head; windows: only these."""
    nwy, nwx = case["H"] // case["wh"], case["W"] // case["ww"]

    def part(side, shift, on, last):
        return ((side - shift) ** 2 + shift ** 2 if on and shift and last else side ** 2)
    total = 0
    for wy in range(nwy):
        for wx in range(nwx):
            if windows is None or wy * nwx + wx in windows:
                total += (part(case["wh"], case["sh"], case["mask"] != "none", wy == nwy - 1)
                          * part(case["ww"], case["sw"], case["mask"] == "swin", wx == nwx - 1))
    return total


def work(case):
    kind = case["kind"]
    if kind in ("attn_fwd", "attn_train", "rope_share"):
        windows = set(_share(case)) if kind == "rope_share" else None
        rows = case["B"] * case["heads"] * (case["H"] * case["W"] if windows is None
                                            else len(windows) * case["wh"] * case["ww"])
        U = case["B"] * case["heads"] * _visible_pairs(case, windows)
        ob, d = (4 if case["out"] == "f32" else 2), case["d"]
        # q, k, v in, o and lse out; training: dO in, dq, dk, dv out (five products backward)
        if kind == "attn_fwd":
            return dict(bytes=rows * (d * (6 + ob) + 4), flops=4 * d * U)
        return dict(bytes=rows * (d * (8 + 4 * ob) + 4), flops=14 * d * U)
    if kind == "layer":
        C, hidden = case["heads"] * case["d"], case["hidden"]
        N = case["B"] * case["H"] * case["W"]
        weights = C * (4 * C + 3 * hidden)
        return dict(bytes=N * C * 2 * 4 + weights * (2 + 4),
                    flops=6 * N * weights + 14 * case["d"] * case["B"] * case["heads"] * _visible_pairs(case))
    if kind == "proj_fwd":
        N, C, hidden = case["samples"] * case["rows"], case["C"], case["hidden"]
        return dict(bytes=2 * (N * (C + hidden) + C * (4 * C + 3 * hidden) + N * (5 * C + hidden)),
                    flops=2 * N * C * (4 * C + 3 * hidden))
    if kind == "proj_bwd":
        N, C, F = case["rows"], case["C"], case["F"]
        return dict(bytes=2 * (2 * N * C + N * F + F * C) + 4 * F * C, flops=4 * N * C * F)
    N, C = case["samples"] * case["rows"], case["C"]
    # h <- x; dx <- x, d, y; out <- x, y; dy <- y, d; g <- uv; duv <- uv, dg: each operation's own
    # operands and results (six calls, nothing shared between them)
    return dict(bytes=2 * N * C * (2 + 4 + 3 + 3 + 3 + 5) + 8 * N, flops=40 * N * C)


def tolerance(case):
    """Relative L2 against fp64 on these inputs (largest output), measured, times about four.
    Attention rounds P and dS to bf16 before the second products: 2.4e-3 with bf16 results, 1.7e-3
    to 2.2e-3 with fp32 results.  On blended fields dS cancels and dq inherits the rounding of the
    o that is handed over in bf16: 1.1e-2 to 3.5e-2, of which two implementations share most.
    Projections 2.4e-3 to 3.0e-3, their gradients and the element-wise results 1.7e-3; a whole
    layer hands on nine bf16 tensors, 6.2e-3."""
    kind = case["kind"]
    if kind in ("attn_fwd", "attn_train", "rope_share"):
        if case["data"] == "blend" and case["out"] == "bf16" and kind == "attn_train":
            return {"rel": 3e-2}
        return {"rel": 8e-3 if case["out"] == "f32" else 1e-2}
    return {"rel": {"layer": 2.4e-2, "proj_fwd": 1e-2, "proj_bwd": 7e-3, "layer_ops": 7e-3}[kind]}
