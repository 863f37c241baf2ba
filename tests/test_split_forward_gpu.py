"""The split forward (x W and x W_down as K pieces, then the chain, then the
finishing launch) at ragged rows, columns, K chunks and ranks, on each tile
(32, 64 and 128 x 128, 256 x 128), each piece count (1, 2, 3, 4, 6, 8, 12) and
each finishing kernel that the rule picks, against the fp64 oracle; and the
same call with only the unsplit form's scratch, which must still run.  FORMS
says which form each case runs (tests/test_launches.py holds the rule to it)."""

import numpy as np
import pytest

import oracle
from paper_2603_06492_amd import inputs as inp
from paper_2603_06492_amd import noble

from _parity import TOL, oracle_outputs, row_err
from test_abi import _align, _proj_split

CASES = [
    # id, T, d_in, d_out, r, groups
    ("T1_g3", 1, 1032, 3 * 264, 24, 3),
    ("T1_r8", 1, 264, 72, 8, 1),
    ("T33_r136", 33, 2056, 1000, 136, 1),
    ("T65_g4", 65, 776, 4 * 136, 72, 4),
    ("T129_r64", 129, 1024, 512, 64, 1),
    ("T777_r128", 777, 4104, 1032, 128, 1),
    ("T1601_r256", 1601, 2048, 776, 256, 1),
    ("T401_wide", 401, 4096, 3080, 40, 1),
    # long K: 6 to 12 pieces
    ("T5_deep", 5, 8200, 520, 40, 1),
    ("T33_deep", 33, 8192, 2048, 128, 1),
    ("T1_r128_g3", 1, 4184, 3240, 128, 3),
    ("T1776_deep", 1776, 5584, 152, 104, 1),
    # more finishing workgroups than run at once: the chain and the finish as two launches
    ("T913_r24_g3", 913, 1656, 2040, 24, 3),
    ("T1617_r56_g3", 1617, 2616, 1296, 56, 3),
    ("T199_r72_g3", 199, 1976, 9720, 72, 3),
]
# tile, pieces, finishing kernel (r <= 64 NC in y_finish_kernel<NC>)
FORMS = {
    "T1_g3": ("64x128", 4, "chain_finish"),
    "T1_r8": ("64x128", 1, "chain_finish"),
    "T33_r136": ("32x128", 4, "y_finish<4>"),
    "T65_g4": ("64x128", 3, "chain_finish"),
    "T129_r64": ("64x128", 4, "chain_finish"),
    "T777_r128": ("128x128", 3, "chain_finish"),
    "T1601_r256": ("128x128", 2, "y_finish<4>"),
    "T401_wide": ("128x128", 2, "chain_finish"),
    "T5_deep": ("32x128", 12, "chain_finish"),
    "T33_deep": ("64x128", 8, "chain_finish"),
    "T1_r128_g3": ("64x128", 6, "chain_finish"),
    "T1776_deep": ("128x128", 6, "chain_finish"),
    "T913_r24_g3": ("64x128", 2, "y_finish<1>"),
    "T1617_r56_g3": ("256x128", 2, "y_finish<1>"),
    "T199_r72_g3": ("256x128", 3, "y_finish<2>"),
}
# 3-layer CosNet, whose chain and finish share a launch up to 256 finishing workgroups: id, T, d_in, d_out, r, groups
CASES3 = [
    ("l3_T1401_r8_g2", 1401, 480, 640, 8, 2),
    ("l3_T435_r72_g2", 435, 1096, 2528, 72, 2),
]
FORMS3 = {"l3_T1401_r8_g2": ("64x128", 2, "y_finish<1>"), "l3_T435_r72_g2": ("64x128", 3, "y_finish<2>")}


def _unsplit_scratch(T, di, do, r, G):
    J = G * -(-r // 128)
    S = max(_proj_split(T, di, J), _proj_split(T, do // G, J))
    return _align(T * G * r * 2) + _align(S * T * G * r * 4)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_forward_scratch_of_the_split(case):
    """These shapes are split: the scratch query holds the float32 partials of
    x W_down and x W for the form's pieces."""
    name, T, di, do, r, G = case
    got = noble.noble_linear_fwd_scratch_size(T, di, do, r, noble.NOBLE_BF16, 0, G)
    s = FORMS[name][1]
    assert got == _align(T * G * r * 2) + _align(s * T * G * r * 4) + _align(s * T * do * 4)
    assert got > _unsplit_scratch(T, di, do, r, G)
    res, full = noble.noble_linear_workspace_size(T, di, do, r, noble.NOBLE_BF16, 0, G)
    assert full >= got


@pytest.mark.gpu
@pytest.mark.parametrize("act", ["cos", "tanh", "gelu_m", "cosnet3"])
def test_split_forward_of_other_forms(act):
    """One, two and three applications where the chain and the finish share a launch, H kept."""
    import torch
    from paper_2603_06492_amd.runner import DeviceProblem
    T, di, do, r, G = 40, 1032, 3 * 136, 56, 3
    print(f"[split] {act}", flush=True)
    p = inp.draw_projection("split_" + act, T, di, do, r, "bf16", seed=92, bias_std=0.5, groups=G,
                            layers=noble.layers(act) if act == "cosnet3" else 2)
    dp = DeviceProblem(p, canary=True, activation=act)
    dp.scratch.fill_(255)
    dp.fwd()
    torch.cuda.synchronize()
    assert row_err(dp.y.float().cpu().numpy().astype(np.float64), oracle_outputs(p, activation=act)["y"]) <= TOL["bf16"]
    h = dp.reserve[:4 * T * G * r].view(torch.float32).view(T, G * r).cpu().numpy()
    a = p.arrays
    assert row_err(h, a["x"].astype(np.float64) @ a["W_down"].astype(np.float64)) <= TOL["f32"]
    assert dp.guards_intact(), "write outside an output buffer"


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_split_forward(case):
    import torch
    from paper_2603_06492_amd.runner import DeviceProblem
    name, T, di, do, r, G = case
    print(f"[split] {name}: T={T} d_in={di} d_out={do} r={r} groups={G}", flush=True)
    p = inp.draw_projection(name, T, di, do, r, "bf16", seed=91, bias_std=0.5, groups=G)
    a = p.arrays
    args = [a[k] for k in ("x", "W", "b", "W_down", "omega1", "phi1", "M", "omega2", "phi2", "W_up")]
    ref = oracle.forward_grouped(*args, G)[0] if G > 1 else oracle.forward(*args)[0]
    dp = DeviceProblem(p, canary=True)
    dp.scratch.fill_(255)   # NaN patterns: nothing is read before it is written
    dp.reserve.fill_(255)
    dp.fwd()
    torch.cuda.synchronize()
    y, H = dp.y.float().cpu().numpy().astype(np.float64), dp.reserve.clone()
    assert row_err(y, ref) <= TOL["bf16"]
    assert dp.guards_intact(), "write outside an output buffer"
    # H: float32 sums of x W_down over d_in in any order
    R = G * r
    h = H[:4 * T * R].view(torch.float32).view(T, R).cpu().numpy()
    assert row_err(h, a["x"].astype(np.float64) @ a["W_down"].astype(np.float64)) <= TOL["f32"]
    # the least scratch of a forward: the unsplit form, same results to rounding
    dp.scratch = dp.scratch[:_unsplit_scratch(T, di, do, r, G)].contiguous()
    dp.y.fill_(float("nan"))
    dp.fwd()
    torch.cuda.synchronize()
    y1 = dp.y.float().cpu().numpy().astype(np.float64)
    assert row_err(y1, ref) <= TOL["bf16"]
    dp.scratch = dp.scratch[:-256].contiguous()
    with pytest.raises(noble.NobleError):
        dp.fwd()


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES3, ids=[c[0] for c in CASES3])
def test_split_forward_of_the_3_layer_form_in_two_launches(case):
    import torch
    from paper_2603_06492_amd.runner import DeviceProblem
    name, T, di, do, r, G = case
    print(f"[split] {name}: T={T} d_in={di} d_out={do} r={r} groups={G}", flush=True)
    p = inp.draw_projection(name, T, di, do, r, "bf16", seed=93, bias_std=0.5, groups=G, layers=3)
    dp = DeviceProblem(p, canary=True, activation="cosnet3")
    dp.scratch.fill_(255)
    dp.fwd()
    torch.cuda.synchronize()
    ref = oracle_outputs(p, activation="cosnet3")["y"]
    assert row_err(dp.y.float().cpu().numpy().astype(np.float64), ref) <= TOL["bf16"]
    assert dp.guards_intact(), "write outside an output buffer"


@pytest.mark.gpu
@pytest.mark.parametrize("case", [c for c in CASES if c[5] == 1], ids=[c[0] for c in CASES if c[5] == 1])
def test_zero_up_projection(case):
    """W_up = 0 against the plain layer.  The unsplit form and one K piece add the products in the plain layer's order:
    y is equal bit for bit.  More pieces add the same float32 products in another order, and then round to bf16 once,
    as the plain layer does."""
    import torch
    from paper_2603_06492_amd.runner import DeviceProblem
    name, T, di, do, r, G = case
    print(f"[split] W_up = 0, {name}", flush=True)
    p = inp.draw_projection(name, T, di, do, r, "bf16", seed=94, bias_std=0.5)
    p.arrays["W_up"][:] = 0
    a, b = DeviceProblem(p), DeviceProblem(p, branch=False)
    a.fwd()
    b.fwd()
    torch.cuda.synchronize()
    ya, yb = a.y.float(), b.y.float()
    if FORMS[name][1] == 1:
        assert bool((ya == yb).all())
    else:
        # a sum of d_in + 1 float32 terms in any order is within (d_in + 1) 2^-24 sum |terms| of the exact one; rounding
        # to bf16 adds 2^-8 of the value on either side
        x, W, bias = (torch.from_numpy(p.arrays[k].astype(np.float64)) for k in ("x", "W", "b"))
        terms = x.abs() @ W.abs() + bias.abs()
        bound = (2 * (di + 1) * 2.0 ** -24 * terms).to(ya.device) + 2.0 ** -8 * (ya.abs() + yb.abs()).double()
        assert bool(((ya - yb).abs() <= bound).all())
    a.scratch = a.scratch[:_unsplit_scratch(T, di, do, r, G)].contiguous()
    a.y.fill_(float("nan"))
    a.fwd()
    torch.cuda.synchronize()
    assert bool((a.y.float() == yb).all())
