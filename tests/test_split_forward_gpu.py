"""The split forward (x W and x W_down as K pieces, then the chain, then the
finishing launch) at ragged rows, columns, K chunks and ranks, on each tile
and piece count the rule picks, against the fp64 oracle; and the same call with
only the unsplit form's scratch, which must still run."""

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
    # 6 to 12 pieces, 32 x 128 tiles
    ("T5_deep", 5, 8200, 520, 40, 1),
    ("T33_deep", 33, 8192, 2048, 128, 1),
]


def _unsplit_scratch(T, di, do, r, G):
    J = G * -(-r // 128)
    S = max(_proj_split(T, di, J), _proj_split(T, do // G, J))
    return _align(T * G * r * 2) + _align(S * T * G * r * 4)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_forward_scratch_of_the_split(case):
    """These shapes are split: the scratch query holds the float32 partials of
    x W_down and x W for 1 to 12 pieces."""
    _, T, di, do, r, G = case
    got = noble.noble_linear_fwd_scratch_size(T, di, do, r, noble.NOBLE_BF16, 0, G)
    sizes = [_align(T * G * r * 2) + _align(s * T * G * r * 4) + _align(s * T * do * 4) for s in (1, 2, 3, 4, 6, 8, 12)]
    assert got in sizes and got > _unsplit_scratch(T, di, do, r, G)
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
