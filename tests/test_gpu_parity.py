"""GPU parity: the HIP library (through its C ABI) against the fp64 oracle.

Tolerances (bf16 operands, fp32 accumulation): relative L2 <= 5e-3 and
max-abs <= 2e-2 on O, dQ, dK, dV; |LSE error| <= 1e-2.

Outputs delivered in fp32 are held to exactly these numbers.  Outputs delivered in
bf16 carry the rounding of the stored value, which is relative to its magnitude
(8 significant bits: half an ulp is 2^-9 |x|, i.e. 1.6e-2 at |x| = 8): for them the
max-abs bound is scaled by max|ref| / 4 once the reference exceeds 4 in magnitude
(N(0,1) operands give outputs with max |x| of about 4); relative L2 stays 5e-3.
The fp32-output run is the parity figure; the bf16-output run sits beside it.
Every comparison is logged (tests/parity_log.py): test, tensor, output type,
measured rel-L2, max-abs, max|ref| and the bound that was applied.
"""
import numpy as np
import pytest
import torch

from oracle import winattn_oracle as orc
from paper_2509_13523_amd import binding as B
from paper_2509_13523_amd import synth
import parity_log

pytestmark = pytest.mark.gpu

REL_L2, MAX_ABS, LSE_ABS = 5e-3, 2e-2, 1e-2
POLICIES = [B.AERIS_MASK_NONE, B.AERIS_MASK_LAT, B.AERIS_MASK_SWIN]


def to_dev(bits):
    return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)


def to_f64(t):
    return t.float().cpu().numpy().astype(np.float64)


def check(name, got, ref, bf16_out, bound=None):
    """bound: optional element-wise allowance subtracted from the error before the max-abs test
    (see operand_rounding_bounds); relative L2 is never widened."""
    got = to_f64(got) if isinstance(got, torch.Tensor) else got
    assert np.isfinite(got).all(), name
    # a one-token window has dQ = dK = 0 exactly: allow an absolute floor of 1e-5 per element
    nref = max(np.linalg.norm(ref), 2e-3 * np.sqrt(ref.size))
    rel = np.linalg.norm(got - ref) / nref
    err = np.abs(got - ref)
    max_ref = np.abs(ref).max()
    tol = MAX_ABS * (max(1.0, max_ref / 4.0) if bf16_out else 1.0)
    parity_log.add(name, "bf16" if bf16_out else "f32", rel, err.max(), max_ref, tol,
                   None if bound is None else np.linalg.norm(bound) / nref)
    assert rel <= REL_L2, "%s rel_l2 %.3e" % (name, rel)
    excess = err if bound is None else np.maximum(err - bound, 0.0)
    assert excess.max() <= tol, "%s max_abs %.3e > %.3e" % (name, excess.max(), tol)


def operand_rounding_bounds(qw, kw, vw, dow, reg, scale):
    """First-order bounds, per element, on what the kernels' rounding of P and dS to bf16 before
    the second products does to O, dV, dQ, dK of one (batch, window, head).  Every element of P
    or dS moves by at most half an ulp, u = 2^-8 relative, so
        |d O|  <= u P |V|,            |d dV| <= u P^T |dO|,
        |d delta_i| <= e_i = sum_c |dO_ic| (u P |V|)_ic      (delta is formed from the kernel's O),
        |d dQ| <= scale (u |dS| |K| + e_i |sum_j P_ij K_j|),
        |d dK| <= scale (u |dS|^T |Q| + sum_i P_ij e_i |Q_i|),
    with P, dS from the oracle.  Where operands are far from unit scale and the sums cancel these
    exceed any fixed absolute bound (an fp64 emulation of exactly these roundings reproduces the
    GPU's errors on such data)."""
    u = 2.0 ** -8
    _, _, P = orc.window_pair_fwd(qw, kw, vw, reg, scale)
    out = {"o": u * (P @ np.abs(vw))}
    if dow is not None:
        dP = dow @ vw.T
        dS = np.abs(P * (dP - (P * dP).sum(axis=1)[:, None]))
        e = (np.abs(dow) * out["o"]).sum(axis=1)
        out["dv"] = u * (P.T @ np.abs(dow))
        out["dq"] = scale * (u * (dS @ np.abs(kw)) + e[:, None] * np.abs(P @ kw))
        out["dk"] = scale * (u * (dS.T @ np.abs(qw)) + (P * e[:, None]).T @ np.abs(qw))
    return out


def check_lse(got, ref, rel=0.0):
    got = to_f64(got) if isinstance(got, torch.Tensor) else got
    err = np.abs(got - ref)
    parity_log.add("lse", "f32", np.linalg.norm(err) / np.linalg.norm(ref), err.max(),
                   np.abs(ref).max(), LSE_ABS)
    assert (err <= LSE_ABS + rel * np.abs(ref)).all()


def handover_bounds(qw, kw, vw, dow, reg, scale):
    """First-order bounds on the change of dQ, dK of one (batch, window, head) when
    delta = sum_c dO*O is formed from O stored in bf16 (one ulp, 2^-8 relative, per
    element): |d dQ_i| <= scale e_i |sum_j P_ij K_j|, |d dK_j| <= scale sum_i P_ij e_i |Q_i|,
    e_i = 2^-8 sum_c |dO_ic||O_ic|.  P and O come from the oracle."""
    O, _, P = orc.window_pair_fwd(qw, kw, vw, reg, scale)
    e = 2.0 ** -8 * (np.abs(dow) * np.abs(O)).sum(axis=1)
    return scale * e[:, None] * np.abs(P @ kw), scale * (P * e[:, None]).T @ np.abs(qw)


def check_with_bound(name, got, ref, bound):
    """bf16 outputs: the plain tolerance plus an element-wise first-order bound (the bf16
    hand-over of O, and for far-from-unit-scale operands the operand roundings)."""
    err = np.abs(got - ref)
    assert np.isfinite(got).all(), name
    excess = np.maximum(err - bound, 0.0)
    max_ref = np.abs(ref).max()
    tol = MAX_ABS * max(1.0, max_ref / 4.0)
    nref = np.linalg.norm(ref)
    parity_log.add(name, "bf16", np.linalg.norm(err) / nref, err.max(), max_ref, tol,
                   np.linalg.norm(bound) / nref)
    assert excess.max() <= tol, "%s max_abs excess %.3e > %.3e" % (name, excess.max(), tol)
    assert np.linalg.norm(err) <= REL_L2 * nref + np.linalg.norm(bound), name


def run_case(shape, win, shift, mask, kind="normal", seed=1, bwd=True, scale=None,
             outs=(B.AERIS_DT_F32, B.AERIS_DT_BF16)):
    bits = synth.make_inputs(kind, seed, shape, 4)
    q64, k64, v64, do64 = [synth.bf16_bits_to_f64(b) for b in bits]
    tq, tk, tv, tdo = [to_dev(b) for b in bits]
    o_ref, lse_ref = orc.winattn_fwd(q64, k64, v64, win, shift, mask, scale)
    if bwd:
        dq_ref, dk_ref, dv_ref, _ = orc.winattn_bwd(q64, k64, v64, do64, win, shift, mask, scale)
    for out in outs:
        bf = out == B.AERIS_DT_BF16
        o, lse = B.aeris_winattn_fwd(tq, tk, tv, win, shift, mask, scale, out_dtype=out)
        torch.cuda.synchronize()
        check("o", o, o_ref, bf)
        check_lse(lse, lse_ref)
        if bwd:
            dq, dk, dv = B.aeris_winattn_bwd(tq, tk, tv, o, lse, tdo, win, shift, mask, scale,
                                             out_dtype=out)
            torch.cuda.synchronize()
            check("dq", dq, dq_ref, bf)
            check("dk", dk, dk_ref, bf)
            check("dv", dv, dv_ref, bf)


# ---- BASELINE config 1: tiny grid, 8x8 windows ------------------------------------------
@pytest.mark.parametrize("mask", POLICIES)
@pytest.mark.parametrize("shift", [(0, 0), (4, 4)])
def test_config1_tiny(mask, shift):
    run_case((1, 64, 128, 4, 32), (8, 8), shift, mask, seed=1001)


# ---- BASELINE config 2: 1-degree-class grid, 12x12 windows, fwd+bwd ---------------------
@pytest.mark.parametrize("kind", ["normal", "smooth"])
@pytest.mark.parametrize("shift", [(0, 0), (6, 6)])
def test_config2_one_degree(kind, shift):
    run_case((1, 180, 360, 8, 64), (12, 12), shift, B.AERIS_MASK_SWIN, kind=kind, seed=2001,
             outs=(B.AERIS_DT_F32,) if kind == "smooth" else (B.AERIS_DT_F32, B.AERIS_DT_BF16))


def test_config2_smooth_bf16_handover():
    """Smooth fields give peaked softmax rows, where dS = P o (dP - delta) cancels
    almost completely.  When the forward output is handed to the backward pass in
    bf16, delta = sum_c dO*O inherits O's storage rounding (up to one bf16 ulp,
    2^-8 relative, per element), which does not cancel.  dQ and dK are therefore
    held to the plain tolerance plus the first-order effect of that perturbation,
        |d dQ_i| <= scale * e_i * |sum_j P_ij K_j|,  |d dK_j| <= scale * sum_i P_ij e_i |Q_i|,
        e_i = 2^-8 * sum_c |dO_ic| |O_ic|,
    evaluated with the oracle's P; O, LSE and dV keep the plain tolerance."""
    shape, win, shift, mask = (1, 180, 360, 8, 64), (12, 12), (6, 6), B.AERIS_MASK_SWIN
    Bn, H, W, nh, d = shape
    scale = 1.0 / np.sqrt(d)
    bits = synth.make_inputs("smooth", 2001, shape, 4)
    q64, k64, v64, do64 = [synth.bf16_bits_to_f64(b) for b in bits]
    tq, tk, tv, tdo = [to_dev(b) for b in bits]
    o_ref, lse_ref = orc.winattn_fwd(q64, k64, v64, win, shift, mask)
    dq_ref, dk_ref, dv_ref, _ = orc.winattn_bwd(q64, k64, v64, do64, win, shift, mask)
    bq, bk = np.zeros_like(q64), np.zeros_like(q64)
    for wy in range(H // win[0]):
        for wx in range(W // win[1]):
            y, x, yh, xh = orc.window_tokens(H, W, win, shift, wy, wx)
            reg = orc.token_regions(H, W, win, shift, mask, yh, xh)
            for h in range(nh):
                bq[0, y, x, h], bk[0, y, x, h] = handover_bounds(
                    q64[0, y, x, h], k64[0, y, x, h], v64[0, y, x, h], do64[0, y, x, h], reg, scale)
    o, lse = B.aeris_winattn_fwd(tq, tk, tv, win, shift, mask)
    dq, dk, dv = B.aeris_winattn_bwd(tq, tk, tv, o, lse, tdo, win, shift, mask)
    torch.cuda.synchronize()
    check("o", o, o_ref, True)
    check("dv", dv, dv_ref, True)
    check_lse(lse, lse_ref)
    check_with_bound("dq", to_f64(dq), dq_ref, bq)
    check_with_bound("dk", to_f64(dk), dk_ref, bk)


# ---- several resident tiles, ragged tails, every head_dim and policy --------------------
@pytest.mark.parametrize("mask", POLICIES)
@pytest.mark.parametrize("d", [32, 64, 128])
def test_ragged_multi_tile(mask, d):
    # T = 400 = 3*128 + 16 (ragged resident tile), 6*64 + 16 (ragged streamed tile)
    run_case((1, 40, 60, 2, d), (20, 20), (10, 10), mask, kind="blend", seed=30 + d)


@pytest.mark.parametrize("mask", POLICIES)
def test_six_hour_model_windows(mask):
    # 30x30 windows, shift 15: T = 900 is not a multiple of 16
    run_case((1, 60, 90, 2, 128), (30, 30), (15, 15), mask, seed=41)


@pytest.mark.parametrize("win,shift", [((1, 1), (0, 0)), ((2, 2), (1, 1)), ((4, 4), (2, 1)),
                                       ((5, 3), (2, 2)), ((6, 10), (2, 3))])
def test_small_and_non_square_windows(win, shift):
    H, W = win[0] * 4, win[1] * 6
    run_case((2, H, W, 3, 64), win, shift, B.AERIS_MASK_SWIN, seed=51)


@pytest.mark.parametrize("shape,win", [
    ((1, 31, 11, 5, 32), (31, 1)),        # 31 tokens: pairs dealt one by one
    ((1, 8, 44, 5, 32), (8, 4)),          # 32 tokens: eight windows dealt whole, three pair by pair
    ((3, 16, 24, 3, 128), (8, 8)),        # 18 windows over three batch members
    ((1, 16, 360, 3, 64), (16, 40)),      # 640 tokens, nine windows
    ((1, 16, 369, 2, 64), (16, 41)),      # 656 tokens: pairs dealt one by one again
])
def test_every_pair_has_one_workgroup(shape, win):
    """Both ways of dealing (window, head) pairs to workgroups, at their edges and remainders."""
    run_case(shape, win, (win[0] // 2, win[1] // 2), B.AERIS_MASK_SWIN, seed=55)


@pytest.mark.parametrize("heads,d,win", [
    (2, 32, (31, 1)), (2, 32, (8, 4)),        # held whole, few bytes: pairs dealt one by one
    (2, 32, (13, 3)), (3, 32, (8, 5)),
    (3, 32, (12, 16)), (3, 32, (1, 193)),     # 192 tokens held whole, 193 streamed
    (3, 32, (16, 16)), (3, 32, (13, 20)),     # up to 256: the forward kernel
    (2, 32, (24, 24)), (2, 32, (20, 29)),     # up to 576: the others
    (1, 32, (8, 8)), (1, 32, (14, 14)),       # one head: never
    (16, 32, (8, 8)), (16, 32, (14, 14)),
    (8, 64, (5, 7)), (8, 64, (6, 6)),
    (8, 64, (8, 12)), (8, 64, (1, 97)),       # rows of a multiple of 1 KB: forward streamed from 97 to 128
    (8, 64, (8, 16)), (8, 64, (3, 43)),
    (8, 64, (12, 12)), (8, 64, (5, 29)),      # 144, backward streamed from 145
    (8, 64, (12, 16)), (8, 64, (1, 193)),     # 192, both streamed from 193
    (8, 64, (20, 20)), (8, 64, (18, 23)),     # up to 400: the forward kernel
    (8, 64, (28, 28)), (8, 64, (28, 29)),     # up to 784: the others
    (4, 128, (8, 16)), (4, 128, (43, 3)),     # from 129 tokens
    (4, 128, (28, 28)), (4, 128, (28, 29)),   # up to 784
])
def test_whole_windows_dealt_to_an_xcd(heads, d, win):
    """The edges of the ranges in which the streamed kernels have whole windows, eight of these nine, dealt to
    XCDs, and of the windows that reach those kernels at all."""
    run_case((1, win[0], win[1] * 9, heads, d), win, (win[0] // 2, win[1] // 2), B.AERIS_MASK_SWIN, seed=57)


@pytest.mark.parametrize("shape,win", [
    ((1, 183, 180, 3, 32), (3, 4)),         # from 12 tokens the forward kernel too, 2744 windows of 2745
    ((1, 183, 180, 3, 32), (3, 3)),         # from 9 the backward kernel, 3656 of 3660
    ((3, 104, 104, 3, 32), (13, 8)),        # 104 tokens, 312 windows over three batch members
    ((1, 104, 40, 3, 32), (13, 8)),         # bytes below the line: pairs dealt one by one
    ((1, 120, 429, 16, 64), (8, 13)),       # 495 windows, backward kernel (forward streamed)
])
def test_whole_short_windows_dealt_to_an_xcd(shape, win):
    """Windows and heads held whole: dealt to XCDs by windows where windows and bytes are above the lines.
    With fp32 results: the rounding of a bf16 O on its way to delta, |d dQ_i| <= scale e_i |sum_j P_ij K_j| (see
    test_config2_smooth_bf16_handover), is not part of the plain tolerance, and among the 53 million elements of
    the last case one comes to 2.08e-2."""
    run_case(shape, win, (win[0] // 2, win[1] // 2), B.AERIS_MASK_SWIN, seed=59, outs=(B.AERIS_DT_F32,))


@pytest.mark.parametrize("shape,win,kernel", [
    ((1, 16, 16, 3, 32), (8, 8), 0),          # 64 tokens: one kernel for all three gradients
    ((1, 26, 15, 3, 32), (13, 5), 0),
    ((1, 104, 160, 3, 32), (13, 5), 0),
    ((1, 104, 170, 3, 32), (13, 5), 0),
    ((1, 28, 42, 3, 32), (14, 14), 1),        # 196 tokens, 48 workgroups
    ((1, 112, 224, 3, 32), (14, 14), 1),      # 768
    ((1, 112, 238, 3, 32), (14, 14), 2),      # 816
    ((1, 160, 260, 2, 32), (20, 20), 2),      # 400 tokens, 832
])
def test_head_dim_32_dkdv_by_window_and_grid_size(shape, win, kernel):
    """Both orders of reads of the dK/dV kernel, at the edges of their rule, and the windows below it."""
    shift = (win[0] // 2, win[1] // 2)
    assert B.aeris_winattn_plan(B.make_params(shape, win, shift, B.AERIS_MASK_SWIN))[1] == kernel
    run_case(shape, win, shift, B.AERIS_MASK_SWIN, seed=58)


@pytest.mark.parametrize("win", [(2, 2), (12, 16), (13, 15), (28, 64), (33, 55)])
def test_head_dim_128_dkdv_by_window_size(win):
    """Up to 1792 tokens the generic dK/dV kernel; 1815: the software-pipelined one."""
    run_case((1, win[0] * 2, win[1] * 3, 2, 128), win, (win[0] // 2, win[1] // 2), B.AERIS_MASK_SWIN,
             seed=56)


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("win", [(1, 1), (3, 5), (4, 4), (1, 17), (4, 8), (3, 11), (6, 8), (7, 7), (7, 9),
                                 (8, 8), (5, 13), (8, 16), (3, 43), (12, 12), (5, 29), (11, 16), (12, 16),
                                 (1, 193)])
def test_short_windows_by_size(win, d):
    """Windows around the units of 16 keys, blocks of 32 queries and one to four waves of the one-kernel
    backward pass, and on both sides of where it ends (192, 144, 64 tokens at head_dim 32, 64, 128);
    the statistics it leaves serve a dK/dV stage of its own."""
    shape, shift = (1, 2 * win[0], 3 * win[1], 2, d), (win[0] // 2, win[1] // 3)
    run_case(shape, win, shift, B.AERIS_MASK_SWIN, seed=77)
    tq, tk, tv, tdo = [to_dev(b) for b in synth.make_inputs("normal", 78, shape, 4)]
    o, lse = B.aeris_winattn_fwd(tq, tk, tv, win, shift, B.AERIS_MASK_LAT)
    ws = torch.empty(B.aeris_winattn_bwd_workspace_bytes(B.make_params(shape, win, shift, B.AERIS_MASK_LAT)),
                     dtype=torch.uint8, device="cuda")
    whole, again = [[torch.full_like(tq, float("nan")) for _ in range(3)] for _ in range(2)]
    for g, stages in ((whole, B.AERIS_BWD_ALL), (again, B.AERIS_BWD_DKDV)):
        B.aeris_winattn_bwd_stages(tq, tk, tv, o, lse, tdo, win, shift, B.AERIS_MASK_LAT, dq=g[0], dk=g[1],
                                   dv=g[2], workspace=ws, stages=stages)
    torch.cuda.synchronize()
    for a, b in zip(whole[1:], again[1:]):
        assert torch.equal(a, b)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("win,shift,d,clean,poisoned", [
    ((9, 16), 3, 32, 96, 128),     # regions of 96 and 48 tokens: a window and head whole in a workgroup
    ((9, 16), 3, 64, 96, 128),
    ((12, 16), 6, 32, 96, 128),    # 96 and 96
    ((12, 16), 6, 64, 96, 128),    # forward whole, backward streamed
    ((8, 16), 4, 32, 64, 64),      # 64 and 64
    ((8, 16), 4, 64, 64, 64),      # forward streamed, backward whole
    ((8, 16), 4, 128, 64, 64),     # forward whole, backward streamed
    ((4, 16), 2, 128, 32, 32),     # 32 and 32
    ((16, 16), 8, 64, 128, 128),   # streamed
    ((16, 16), 8, 128, 128, 128),
])
def test_nonfinite_tokens_do_not_reach_other_mask_regions(win, shift, d, clean, poisoned, value):
    """Masked pairs of tokens are left out in blocks, not multiplied by zero: tokens from `poisoned` on that
    are not finite change nothing for the first `clean` tokens of their window, which another mask region
    holds (the two share no block), and nothing in other windows."""
    nh, mask, shift = 3, B.AERIS_MASK_LAT, (shift, 0)
    H, W = 2 * win[0], 3 * win[1]
    shape = (1, H, W, nh, d)
    good = [to_dev(b) for b in synth.make_inputs("normal", 79, shape, 4)]
    at = torch.arange(win[0] * win[1], device="cuda").view(win)      # tokens of a window of the last row,
    at = torch.cat([torch.full((win[0], W), -1, device="cuda"), at.repeat(1, 3)])    # in the shifted frame
    at = torch.roll(at, shift[0], 0)
    bad, keep = at >= poisoned, at < clean
    poison = []
    for t in good:
        t = t.clone()
        t[:, bad] = value
        poison.append(t)
    runs = []
    for q, k, v, do in (good, poison):
        o, lse = B.aeris_winattn_fwd(q, k, v, win, shift, mask)
        runs.append([o, lse.permute(0, 2, 3, 1), *B.aeris_winattn_bwd(q, k, v, o, lse, do, win, shift, mask)])
    torch.cuda.synchronize()
    for name, a, b in zip(("o", "lse", "dq", "dk", "dv"), *runs):
        assert torch.isfinite(a.float()).all(), name
        assert torch.equal(a[:, keep], b[:, keep]), name


@pytest.mark.parametrize("shift", [(0, 0), (5, 7)])
def test_one_window_is_global_attention(shift):
    run_case((1, 24, 40, 2, 64), (24, 40), shift, B.AERIS_MASK_NONE, seed=61)
    run_case((1, 24, 40, 2, 64), (24, 40), shift, B.AERIS_MASK_SWIN, seed=62)


@pytest.mark.parametrize("shift", [(7, 3), (1, 19)])
def test_arbitrary_shift(shift):
    run_case((1, 40, 60, 1, 64), (20, 20), shift, B.AERIS_MASK_SWIN, seed=71)


def test_softmax_scale_override_and_peaked_rows():
    # 1.5 times the default scale at d=64
    run_case((1, 16, 32, 2, 64), (16, 16), (8, 8), B.AERIS_MASK_LAT, scale=0.18, seed=81)


@pytest.mark.parametrize("d", [64, 128])
def test_paper_window_60x60(d):
    # two 60x60 windows (T = 3600) of the 24-hour model, seam + corner regions
    run_case((1, 60, 120, 2, d), (60, 60), (30, 30), B.AERIS_MASK_SWIN, kind="blend", seed=91,
             outs=(B.AERIS_DT_BF16,))


@pytest.mark.parametrize("d", [64, 128])
def test_windows_between_the_narrow_and_wide_forward_tiles(d):
    # T = 2500 (50x50): forward tiles of 256 queries with a ragged tenth tile of 196;
    # T = 2025 (45x45) stays on tiles of 128
    run_case((1, 50, 100, 1, d), (50, 50), (25, 25), B.AERIS_MASK_SWIN, seed=93,
             outs=(B.AERIS_DT_BF16,))
    run_case((1, 45, 45, 1, d), (45, 45), (20, 11), B.AERIS_MASK_LAT, seed=94, bwd=False,
             outs=(B.AERIS_DT_F32,))


def test_config5_unshifted_layer_fwd_bwd_sampled():
    # the other layer of the bench step: shift 0 (no seam, no mask effect)
    samples = [(0, 2, 9, 5), (1, 0, 0, 3), (2, 6, 17, 12), (3, 11, 20, 0)]
    sampled_check((4, 720, 1440, 16, 128), (60, 60), (0, 0), B.AERIS_MASK_SWIN, "blend", 5001,
                  True, samples, sigmas=[0.1, 0.5, 1.0, 2.0])


@pytest.mark.parametrize("d", [64, 128])
def test_maximum_window_tokens(d):
    # one 64 x 128 window = 8192 tokens, the largest the on-chip token table holds; shifted, so the
    # window splits into four mask regions of 2048 tokens
    run_case((1, 64, 128, 1, d), (64, 128), (32, 64), B.AERIS_MASK_SWIN, kind="blend", seed=95,
             outs=(B.AERIS_DT_BF16,))


@pytest.mark.parametrize("d,win,windows,plan", [
    (64, (12, 12), (2, 2), (3, 0)),       # window and head whole, forward and backward; three share the queries
    (32, (9, 16), (2, 3), (3, 0)),
    (128, (8, 8), (2, 3), (1, 0)),
    (64, (10, 10), (2, 3), (0, 0)),       # forward streamed
    (32, (14, 14), (2, 3), (0, 1)),       # streamed; dK/dV with its operands read first
    (64, (14, 17), (2, 3), (0, 1)),       # dQ of 238 tokens: a second, partly filled resident tile
    (32, (16, 16), (10, 20), (0, 2)),     # one block ahead
    (128, (9, 9), (2, 3), (2, 2)),        # dK/dV one block ahead, forward whole
    (128, (17, 17), (2, 3), (0, 2)),
    (128, (33, 55), (1, 2), (0, 3)),      # 1815 tokens: pipelined
    (64, (46, 45), (1, 2), (0, 1)),       # 2070: forward tiles of 256 queries
    (128, (46, 45), (2, 1), (0, 3)),
])
def test_packed_qkv_strides(d, win, windows, plan):
    """Queries, keys and values interleaved per token, and their gradients in the same packing, in every
    kernel that a window can take: a row of a token is three times as far
    from the next as its heads are, and each kernel makes these addresses for itself."""
    shape, shift, mask = (1, win[0] * windows[0], win[1] * windows[1], 2, d), (win[0] // 2, win[1] // 2), B.AERIS_MASK_SWIN
    Bn, H, W, nh, d = shape
    bits = synth.make_inputs("normal", 5, shape, 4)
    q64, k64, v64, do64 = [synth.bf16_bits_to_f64(b) for b in bits]
    packed = torch.stack([to_dev(b) for b in bits[:3]], dim=3).contiguous()   # [B,H,W,3,nh,d]
    dpacked = torch.full_like(packed, float("nan"))
    tdo = to_dev(bits[3])
    o = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((Bn, nh, H, W), dtype=torch.float32, device="cuda")
    p = B.make_params(shape, win, shift, mask, qkv_strides=(3 * nh * d, d))
    assert B.aeris_winattn_plan(p) == plan
    import ctypes
    lib = B.load()
    esz = 2
    ptr = lambda t, i: t.data_ptr() + i * nh * d * esz
    stream = torch.cuda.current_stream().cuda_stream
    rc = lib.aeris_winattn_fwd(ctypes.byref(p), ptr(packed, 0), ptr(packed, 1), ptr(packed, 2),
                               o.data_ptr(), lse.data_ptr(), stream)
    assert rc == 0
    ws = torch.empty(B.aeris_winattn_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    rc = lib.aeris_winattn_bwd(ctypes.byref(p), ptr(packed, 0), ptr(packed, 1), ptr(packed, 2),
                               o.data_ptr(), lse.data_ptr(), tdo.data_ptr(), ptr(dpacked, 0),
                               ptr(dpacked, 1), ptr(dpacked, 2), ws.data_ptr(), ws.numel(), stream)
    assert rc == 0
    torch.cuda.synchronize()
    o_ref, _ = orc.winattn_fwd(q64, k64, v64, win, shift, mask)
    dq_ref, dk_ref, dv_ref, _ = orc.winattn_bwd(q64, k64, v64, do64, win, shift, mask)
    check("o", o, o_ref, True)
    for i, ref in enumerate((dq_ref, dk_ref, dv_ref)):
        check("d%d" % i, dpacked[:, :, :, i], ref, True)


def test_backward_is_bitwise_reproducible_and_staged_equals_whole():
    shape, win, shift, mask = (1, 40, 60, 2, 128), (20, 20), (10, 10), B.AERIS_MASK_SWIN
    tq, tk, tv, tdo = [to_dev(b) for b in synth.make_inputs("normal", 9, shape, 4)]
    o, lse = B.aeris_winattn_fwd(tq, tk, tv, win, shift, mask)
    a = B.aeris_winattn_bwd(tq, tk, tv, o, lse, tdo, win, shift, mask)
    b = B.aeris_winattn_bwd(tq, tk, tv, o, lse, tdo, win, shift, mask)
    ws = torch.empty(B.aeris_winattn_bwd_workspace_bytes(B.make_params(shape, win, shift, mask)),
                     dtype=torch.uint8, device="cuda")
    c = [torch.zeros_like(tq) for _ in range(3)]
    for st in (B.AERIS_BWD_DELTA, B.AERIS_BWD_DKDV, B.AERIS_BWD_DQ):
        B.aeris_winattn_bwd_stages(tq, tk, tv, o, lse, tdo, win, shift, mask, dq=c[0], dk=c[1],
                                   dv=c[2], workspace=ws, stages=st)
    torch.cuda.synchronize()
    for x, y, z in zip(a, b, c):
        assert torch.equal(x.view(torch.int16), y.view(torch.int16))
        assert torch.equal(x.view(torch.int16), z.view(torch.int16))


@pytest.mark.parametrize("d,win", [(32, (4, 4)), (32, (6, 7)), (32, (12, 16)), (32, (14, 14)), (64, (1, 9)), (64, (8, 8)),
                                   (64, (12, 12)), (64, (5, 29)), (128, (5, 5)), (128, (8, 8)), (128, (5, 13))])
@pytest.mark.parametrize("out", [B.AERIS_DT_BF16, B.AERIS_DT_F32])
def test_any_order_of_stages_equals_the_whole(d, win, out):
    """Every selection of stages, in any order after the statistics, gives the bits of the whole backward call,
    leaves the outputs of the others alone and leaves the same statistics, on both sides of the window
    size from which one kernel makes all three gradients."""
    shape, shift, mask = (2, 2 * win[0], 3 * win[1], 2, d), (win[0] // 2, win[1] // 3), B.AERIS_MASK_SWIN
    tq, tk, tv, tdo = [to_dev(b) for b in synth.make_inputs("normal", 10, shape, 4)]
    o, lse = B.aeris_winattn_fwd(tq, tk, tv, win, shift, mask, out_dtype=out)
    need = B.aeris_winattn_bwd_workspace_bytes(B.make_params(shape, win, shift, mask, None, out))

    def run(*selections):
        ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
        g = [torch.full_like(o, float("nan")) for _ in range(3)]
        for stages in selections:
            B.aeris_winattn_bwd_stages(tq, tk, tv, o, lse, tdo, win, shift, mask, out_dtype=out, dq=g[0], dk=g[1],
                                       dv=g[2], workspace=ws.view(torch.uint8), stages=stages)
        torch.cuda.synchronize()
        return g, ws

    whole, stats = run(B.AERIS_BWD_ALL)
    for selections in ((1, 2, 4), (1, 4, 2), (3, 4), (5, 2), (1, 6), (1,), (3,), (5,)):
        g, ws = run(*selections)
        assert torch.equal(ws, stats), selections
        did = sum(selections) if len(selections) > 1 else selections[0]
        for i, t in enumerate(g):
            if did & (2 if i == 0 else 4):
                assert torch.equal(t, whole[i]), (selections, i)
            else:
                assert torch.isnan(t).all(), (selections, i)


def test_errors_raise_on_gpu_box():
    tq = torch.zeros((1, 16, 16, 1, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.AerisError) as e:
        B.aeris_winattn_fwd(tq, tq, tq, (5, 4), (0, 0))
    assert e.value.code == -3


# ---- full-size workloads (bench launch configuration): sampled pairs + invariants -------
def rows_sum(fn, n_rows, step=48):
    """sum over latitude rows of fn(row slice), in pieces (full-size grids: no whole-tensor
    float64 temporaries)."""
    total = None
    for r0 in range(0, n_rows, step):
        part = fn(slice(r0, min(r0 + step, n_rows)))
        total = part if total is None else total + part
    return total


def sampled_check(shape, win, shift, mask, kind, seed, bwd, samples, sigmas=None,
                  outs=(B.AERIS_DT_F32, B.AERIS_DT_BF16)):
    """Full-size launch: whole-grid invariants plus sampled (batch, window, head) pairs against
    the oracle.  With fp32 outputs everything is held to the plain tolerance; with bf16 outputs
    O reaches the backward pass rounded, and dQ, dK get the plain tolerance plus the
    delta-perturbation bound (see test_config2_smooth_bf16_handover).

    One case needs more: the noise-level-2 ensemble member of config 5.  Its operands have a
    standard deviation of about 2.2 (|V| up to 10, gradients up to 350) and its softmax rows are
    peaked, so the rounding of P and dS to bf16 before the second products (2^-9 relative per
    element; sums that cancel; delta formed from the kernel's own O) moves single elements by
    more than any fixed absolute bound:
    measured with fp32 outputs, O max-abs 2.9e-2 at max|O| = 9.9 and dQ 2.1e-1 at max|dQ| = 35,
    relative L2 1.2e-3 and 3.1e-3.  For members whose noise level exceeds 1 the max-abs test
    therefore allows, element by element, the first-order effect of those two roundings
    (operand_rounding_bounds) on top of the plain 2e-2; relative L2 stays 5e-3.  Every other
    fp32 comparison in this file is held to the plain numbers."""
    Bn, H, W, nh, d = shape
    torch.cuda.empty_cache()
    T = {}     # every device tensor lives here, so a failing check cannot keep them allocated
    try:
        _sampled_check(T, shape, win, shift, mask, kind, seed, bwd, samples, sigmas, outs)
    finally:
        T.clear()
        torch.cuda.empty_cache()


def _sampled_check(T, shape, win, shift, mask, kind, seed, bwd, samples, sigmas, outs):
    Bn, H, W, nh, d = shape
    scale = 1.0 / np.sqrt(d)
    names = ("q", "k", "v", "do") if bwd else ("q", "k", "v")
    T.update(zip(names, synth.make_inputs_device(kind, seed, shape, len(names), sigmas=sigmas)))
    refs, bounds, handover = [], [], []
    for (b, wy, wx, h) in samples:
        sl = lambda t: to_f64(t[b, :, :, h, :])
        res = orc.winattn_pair(sl(T["q"]), sl(T["k"]), sl(T["v"]), sl(T["do"]) if bwd else None,
                               H, W, win, shift, mask, None, wy, wx)
        refs.append(res)
        y, x = res["y"], res["x"]
        qw, kw, vw = sl(T["q"])[y, x], sl(T["k"])[y, x], sl(T["v"])[y, x]
        dow = sl(T["do"])[y, x] if bwd else None
        _, _, yh, xh = orc.window_tokens(H, W, win, shift, wy, wx)
        reg = orc.token_regions(H, W, win, shift, mask, yh, xh)
        wide = sigmas is not None and sigmas[b] > 1.0
        bounds.append(operand_rounding_bounds(qw, kw, vw, dow, reg, scale) if wide else None)
        handover.append(handover_bounds(qw, kw, vw, dow, reg, scale) if bwd else None)
    for out in outs:
        bf = out == B.AERIS_DT_BF16
        T["o"], T["lse"] = B.aeris_winattn_fwd(T["q"], T["k"], T["v"], win, shift, mask,
                                               out_dtype=out)
        if bwd:
            T["dq"], T["dk"], T["dv"] = B.aeris_winattn_bwd(
                T["q"], T["k"], T["v"], T["o"], T["lse"], T["do"], win, shift, mask, out_dtype=out)
        torch.cuda.synchronize()
        assert torch.isfinite(T["o"].view(-1)[:: 997].float()).all()
        # whole-grid properties that hold at any size
        vmin = T["v"].amin(dim=(1, 2)).float()
        vmax = T["v"].amax(dim=(1, 2)).float()
        assert (T["o"].amax(dim=(1, 2)).float() <= vmax + 1e-2).all()
        assert (T["o"].amin(dim=(1, 2)).float() >= vmin - 1e-2).all()
        if bwd:
            for b in range(Bn):
                dsum = lambda t, r: t[b, r].double().sum(dim=(0, 1))
                s_dv = rows_sum(lambda r: dsum(T["dv"], r), H)
                s_do = rows_sum(lambda r: dsum(T["do"], r), H)
                scale_ = rows_sum(lambda r: T["dv"][b, r].double().abs().sum(dim=(0, 1)), H)
                assert ((s_dv - s_do).abs() <= 2e-3 * scale_ + 1e-2).all()
                dot = lambda a, g, r: (a[b, r].double() * g[b, r].double())
                qa = rows_sum(lambda r: dot(T["q"], T["dq"], r).sum(dim=(0, 1, 3)), H)
                kb = rows_sum(lambda r: dot(T["k"], T["dk"], r).sum(dim=(0, 1, 3)), H)
                mag = rows_sum(lambda r: dot(T["q"], T["dq"], r).abs().sum(dim=(0, 1, 3)), H)
                assert ((qa - kb).abs() <= 5e-3 * mag + 1e-2).all()
        for (b, wy, wx, h), res, bnd, hand in zip(samples, refs, bounds, handover):
            sl = lambda t: to_f64(t[b, :, :, h, :])
            y, x = res["y"], res["x"]
            get = lambda name: None if bnd is None else bnd[name]
            check("o", sl(T["o"])[y, x], res["o"], bf, get("o"))
            check_lse(to_f64(T["lse"][b, h])[y, x], res["lse"])
            if not bwd:
                continue
            check("dv", sl(T["dv"])[y, x], res["dv"], bf, get("dv"))
            if bf:
                extra = (0.0, 0.0) if bnd is None else (bnd["dq"], bnd["dk"])
                check_with_bound("dq", sl(T["dq"])[y, x], res["dq"], hand[0] + extra[0])
                check_with_bound("dk", sl(T["dk"])[y, x], res["dk"], hand[1] + extra[1])
            else:
                check("dq", sl(T["dq"])[y, x], res["dq"], False, get("dq"))
                check("dk", sl(T["dk"])[y, x], res["dk"], False, get("dk"))
        for name in ("o", "lse", "dq", "dk", "dv"):
            T.pop(name, None)
        torch.cuda.empty_cache()


def test_config3_quarter_degree_forward_sampled():
    # interior, lat-seam row, lon-seam column, corner; two heads each
    samples = [(0, 3, 7, 0), (0, 3, 7, 9), (0, 11, 5, 1), (0, 11, 5, 15), (0, 4, 23, 2),
               (0, 4, 23, 8), (0, 11, 23, 3), (0, 11, 23, 12)]
    sampled_check((1, 720, 1440, 16, 64), (60, 60), (30, 30), B.AERIS_MASK_SWIN, "normal", 3001,
                  False, samples)


def test_config4_band_share_fwd_bwd_sampled():
    samples = [(0, 0, 4, 0), (0, 0, 23, 7), (0, 1, 9, 13), (0, 1, 23, 23)]
    sampled_check((1, 120, 1440, 24, 128), (60, 60), (30, 30), B.AERIS_MASK_SWIN, "blend", 4001,
                  True, samples)


def test_config5_ensemble_member_fwd_bwd_sampled():
    # exactly the bench workload's launch (B = 4, noise levels 0.1, 0.5, 1.0, 2.0); samples from the
    # smoothest and the noisiest member: interior, corner, lat-seam and lon-seam windows
    samples = [(0, 5, 5, 1), (0, 11, 23, 6), (3, 11, 2, 9), (3, 7, 23, 15)]
    sampled_check((4, 720, 1440, 16, 128), (60, 60), (30, 30), B.AERIS_MASK_SWIN, "blend", 5001,
                  True, samples, sigmas=[0.1, 0.5, 1.0, 2.0])


def test_forward_backward_replay_from_a_hip_graph():
    """The library only launches kernels on the caller's stream (no allocation, no memset, no
    synchronisation), so a forward+backward pair can be captured once and replayed.  Every replay
    must reproduce the eager result bit for bit, with other eager work in between."""
    shape, win, shift, mask = (1, 60, 120, 2, 128), (30, 30), (15, 15), B.AERIS_MASK_SWIN
    Bn, H, W, nh, d = shape
    bits = synth.make_inputs("normal", 97, shape, 4)
    tq, tk, tv, tdo = [to_dev(b) for b in bits]
    o = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((Bn, nh, H, W), dtype=torch.float32, device="cuda")
    grads = [torch.empty_like(o) for _ in range(3)]
    p = B.make_params(shape, win, shift, mask)
    ws = torch.empty(B.aeris_winattn_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")

    def run():
        B.aeris_winattn_fwd(tq, tk, tv, win, shift, mask, o=o, lse=lse)
        B.aeris_winattn_bwd_stages(tq, tk, tv, o, lse, tdo, win, shift, mask, dq=grads[0],
                                   dk=grads[1], dv=grads[2], workspace=ws)

    run()                                   # eager reference (also sets the kernels' LDS limits)
    torch.cuda.synchronize()
    want = [t.clone() for t in (o, lse, *grads)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for rep in range(3):
        for t in (o, lse, *grads):
            t.fill_(float("nan"))           # eager work between the replays
        ws.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in zip((o, lse, *grads), want):
            assert torch.equal(got, ref), rep


def test_seeded_sweep_of_small_shapes():
    """Forty seeded random small problems: window sides from 1 to 24 (ragged tiles, single-token
    windows, non-square windows), any shift including one-axis shifts, every mask policy, every
    head_dim, batch and head counts 1 to 3, default and overridden scale, both output types."""
    rng = np.random.default_rng(20240607)
    for case in range(40):
        wh, ww = int(rng.integers(1, 25)), int(rng.integers(1, 25))
        nwy, nwx = int(rng.integers(1, 4)), int(rng.integers(1, 4))
        sh = int(rng.integers(0, wh)) if rng.random() < 0.8 else 0
        sw = int(rng.integers(0, ww)) if rng.random() < 0.8 else 0
        d = int(rng.choice([32, 64, 128]))
        shape = (int(rng.integers(1, 3)), wh * nwy, ww * nwx, int(rng.integers(1, 4)), d)
        mask = int(rng.choice(POLICIES))
        scale = None if rng.random() < 0.7 else float(rng.uniform(0.05, 0.15))
        out = B.AERIS_DT_F32 if rng.random() < 0.5 else B.AERIS_DT_BF16
        print("case", case, shape, (wh, ww), (sh, sw), mask, scale, out, flush=True)
        run_case(shape, (wh, ww), (sh, sw), mask, kind="normal", seed=7000 + case, scale=scale,
                 outs=(out,))


@pytest.mark.parametrize("d", [32, 128])
def test_very_peaked_rows_exercise_the_running_maximum(d):
    """Scale 16x the default: logits have a standard deviation of 16 and single keys dominate
    their rows, so the lagging running maximum is raised (and the accumulators rescaled) many
    times per row, and most probabilities underflow.  Forward outputs and LSE keep the plain
    tolerance; the LSE bound gets a relative part (|LSE| approaches 100)."""
    shape, win, shift, mask = (1, 32, 64, 2, d), (16, 32), (8, 16), B.AERIS_MASK_SWIN
    scale = 16.0 / np.sqrt(d)
    bits = synth.make_inputs("normal", 99, shape, 3)
    q64, k64, v64 = [synth.bf16_bits_to_f64(b) for b in bits]
    tq, tk, tv = [to_dev(b) for b in bits]
    o_ref, lse_ref = orc.winattn_fwd(q64, k64, v64, win, shift, mask, scale)
    assert np.abs(lse_ref).max() > 50.0
    o, lse = B.aeris_winattn_fwd(tq, tk, tv, win, shift, mask, scale, out_dtype=B.AERIS_DT_F32)
    torch.cuda.synchronize()
    check("o", o, o_ref, False)
    check_lse(lse, lse_ref, rel=1e-5)


@pytest.mark.parametrize("order", ["rising", "falling", "all_low", "late_spike"])
def test_forward_reference_point_under_monotone_and_extreme_logits(order):
    """Logits laid out along the key order so that the forward kernel's reference point has to
    follow them: rising by more than 2^12 per 32-key block (every block overflows the sum test and
    rescales), falling (later blocks underflow against an early maximum), all far below zero
    (nothing may underflow: the first block has to set the reference), and flat with one huge
    logit in the last block.  One window of 512 tokens, d = 32."""
    H, W, d = 8, 64, 32
    T = H * W
    rng = np.random.default_rng(7)
    q = np.zeros((1, H, W, 1, d), dtype=np.float32)
    k = np.zeros_like(q)
    q[..., 0] = 4.0
    j = np.arange(T, dtype=np.float32).reshape(H, W)
    if order == "rising":
        k[0, :, :, 0, 0] = j * 0.5 - 100.0          # logits from -400 to +622 (natural units)
    elif order == "falling":
        k[0, :, :, 0, 0] = 100.0 - j * 0.5
    elif order == "all_low":
        k[0, :, :, 0, 0] = -200.0 + 0.01 * rng.standard_normal((H, W)).astype(np.float32)
    else:
        k[0, :, :, 0, 0] = 0.01 * rng.standard_normal((H, W)).astype(np.float32)
        k[0, H - 1, W - 3, 0, 0] = 150.0
    v = rng.standard_normal(q.shape).astype(np.float32)
    bits = [synth.f32_to_bf16_bits(a) for a in (q, k, v)]
    q64, k64, v64 = [synth.bf16_bits_to_f64(b) for b in bits]
    tq, tk, tv = [to_dev(b) for b in bits]
    o_ref, lse_ref = orc.winattn_fwd(q64, k64, v64, (H, W), (0, 0), B.AERIS_MASK_NONE, 1.0)
    assert np.isfinite(lse_ref).all() and np.abs(lse_ref).max() > 300.0
    o, lse = B.aeris_winattn_fwd(tq, tk, tv, (H, W), (0, 0), B.AERIS_MASK_NONE, 1.0,
                                 out_dtype=B.AERIS_DT_F32)
    torch.cuda.synchronize()
    check("o", o, o_ref, False)
    check_lse(lse, lse_ref, rel=1e-5)
