"""y and dx on each output tile of the bf16 products (64 x 128, 128 x 128,
256 x 128 and 256 x 256), at shapes whose last tiles are ragged in rows and
columns and whose last K chunk of either segment is partly filled, against the
fp64 oracle.  The shapes are those the tile rule sends to each tile: few tiles
(64 x 128), about one wave of 128 x 128 or 256 x 128 tiles where 256 x 256
would leave CUs idle, and full waves of 256 x 256.  TILES and F32_TILES say
which tiles each case runs (tests/test_launches.py holds the rules to them)."""

import pytest

from paper_2603_06492_amd import inputs as inp

from _parity import TOL, oracle_outputs, parity_report

pytestmark = pytest.mark.gpu

CASES = [
    # id, T, d_in, d_out, r, groups
    ("64x128_T1", 1, 72, 136, 8, 1),
    ("64x128_T65", 65, 200, 136, 40, 1),   # y in one K piece, then chain_finish_kernel
    ("64x128_T640_g3", 640, 136, 408, 24, 3),
    ("64x128_T64_exact", 64, 128, 128, 64, 1),
    ("128_T1990", 1990, 2040, 2040, 40, 1),
    ("256x128_T8190", 8190, 1016, 1016, 40, 1),
    ("256_T8190", 8190, 2040, 2040, 72, 1),
    # y: the full wave as 256 x 256 tiles (8192 rows), then the last 258 rows
    ("256_then_64x128_T8450", 8450, 1016, 2040, 40, 1),
    # dx alike; y in three groups
    ("two_launches_T8450_g3", 8450, 2040, 3 * 680, 24, 3),
]
# tiles of y's and of dx's launches
TILES = {
    "64x128_T1": (["64x128"], ["64x128"]),
    "64x128_T65": (["64x128"], ["64x128"]),
    "64x128_T640_g3": (["64x128"], ["64x128"]),
    "64x128_T64_exact": (["64x128"], ["64x128"]),
    "128_T1990": (["128x128"], ["128x128"]),
    "256x128_T8190": (["256x128"], ["256x128"]),
    "256_T8190": (["256x256"], ["256x256"]),
    "256_then_64x128_T8450": (["256x256", "64x128"], ["256x256"]),
    "two_launches_T8450_g3": (["256x256", "128x128"], ["256x256", "64x128"]),
}


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_dense_products_on_every_tile(case):
    from paper_2603_06492_amd.runner import DeviceProblem
    name, T, di, do, r, G = case
    print(f"[tiles] {name}: T={T} d_in={di} d_out={do} r={r} groups={G}", flush=True)
    p = inp.draw_projection(name, T, di, do, r, "bf16", seed=77, bias_std=0.5, groups=G)
    dp = DeviceProblem(p, canary=True)
    dp.fwd()
    dp.bwd()
    rep = parity_report(dp.outputs(), oracle_outputs(p), names=("y", "dx"))
    print(rep, flush=True)
    for k, e in rep.items():
        assert e <= TOL["bf16"], (k, e)
    assert dp.guards_intact(), "write outside an output buffer"


F32_CASES = [
    # id, T, d_in, d_out, r, groups: 64 x 64 tiles below a wave of 128 x 128 ones, 128 x 128 at a full wave
    ("f32_64_T63", 63, 40, 72, 8, 1),
    ("f32_64_T65_g3", 65, 104, 3 * 136, 24, 3),
    ("f32_64_T1030", 1030, 200, 328, 32, 1),
    ("f32_64_T4100", 4100, 1032, 968, 16, 1),   # just past a wave of 128 x 128 tiles: 64 x 64 again
    ("f32_128_T4090", 4090, 1016, 1016, 40, 1),
]
# tiles of y, of dx and of the weight gradients
F32_TILES = {
    "f32_64_T63": ("64x64", "64x64", "64x64"),
    "f32_64_T65_g3": ("64x64", "64x64", "64x64"),
    "f32_64_T1030": ("64x64", "64x64", "64x64"),
    "f32_64_T4100": ("64x64", "64x64", "64x64"),
    "f32_128_T4090": ("128x128", "128x128", "128x128"),
}


@pytest.mark.parametrize("case", F32_CASES, ids=[c[0] for c in F32_CASES])
def test_float32_products_on_both_tiles(case):
    from paper_2603_06492_amd.runner import DeviceProblem
    name, T, di, do, r, G = case
    print(f"[tiles] {name}: T={T} d_in={di} d_out={do} r={r} groups={G}", flush=True)
    p = inp.draw_projection(name, T, di, do, r, "f32", seed=78, bias_std=0.5, groups=G)
    dp = DeviceProblem(p, canary=True)
    dp.fwd()
    dp.bwd()
    rep = parity_report(dp.outputs(), oracle_outputs(p))
    print(rep, flush=True)
    for k, e in rep.items():
        assert e <= TOL["f32"], (k, e)
    assert dp.guards_intact(), "write outside an output buffer"
