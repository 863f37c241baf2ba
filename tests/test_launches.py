"""The launches of libnoble's calls, recorded on the CPU by
tests/c/launch_record.cpp (HIP's launch function replaced, no GPU): what the
launch rules choose, and that every launch can be made."""

import json
import os
import random
import re
import shutil
import subprocess

import pytest

from paper_2603_06492_amd import noble

import bench
import test_split_forward_gpu as split
import test_tiles_gpu as tiles

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2603_06492_amd")
MAX_ITEMS = 2 ** 32 - 1   # work-items of one dispatch along x


@pytest.fixture(scope="session")
def record(tmp_path_factory):
    """record(calls) -> per call (status, [(grid_x, grid_y, block, kernel)], {cleared argument: bytes}); a call is
    (name, T, d_in, d_out, r, dtype, activation, groups[, scratch bytes])."""
    hipcc = next((c for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc"))
                  if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not found")
    noble.lib()   # raises if the library has not been built
    exe = str(tmp_path_factory.mktemp("record") / "launch_record")
    cmd = [hipcc, "-std=c++20", "-O1", "--offload-host-only", "-x", "hip",
           os.path.join(ROOT, "tests", "c", "launch_record.cpp"), "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(PKG, "csrc"), "-L", PKG, "-lnoble", f"-Wl,-rpath,{PKG}", "-rdynamic", "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]

    def run(calls):
        lines = []
        for name, T, di, do, r, dtype, act, G, *scratch in calls:
            dt = {"bf16": noble.NOBLE_BF16, "f32": noble.NOBLE_F32}[dtype]
            lines.append(f"{name} {T} {di} {do} {r} {dt} {noble.activation_code(act)} {G} {scratch[0] if scratch else -1}")
        res = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=600)
        assert res.returncode == 0, res.stderr[-4000:]
        out, launches, zeros = [], [], {}
        for line in res.stdout.splitlines():
            kind, rest = line.split(" ", 1)
            if kind == "launch":
                gx, gy, block, kernel = rest.split(" ", 3)
                launches.append((int(gx), int(gy), int(block), kernel))
            elif kind == "zero":
                arg, n = rest.split()
                zeros[arg] = int(n)
            else:
                out.append((int(rest), launches, zeros))
                launches, zeros = [], {}
        assert len(out) == len(calls)
        return out

    return run


def _oversize(launches):
    return [x for x in launches if x[0] * x[2] > MAX_ITEMS or x[1] > 65535]


# float32, few columns, very many tokens: x and y of 69 GB and 207 GB, which fit a GPU
F32_LONG = [((1 << 30) + 64, 8, 8), (359147193, 8, 136), (359147193, 136, 8), ((1 << 31) - 4096, 8, 8)]


@pytest.mark.parametrize("T,di,do", F32_LONG)
@pytest.mark.parametrize("r", [0, 8])
def test_float32_launches_stay_within_a_dispatch(record, T, di, do, r):
    """What the size query accepts is launched: 64 x 64 tiles only where they fit a dispatch."""
    calls = [(c, T, di, do, r, "f32", "cosnet", 1) for c in ("fwd", "bwd")]
    for st, launches, _ in record(calls):
        assert st == 0 and launches
        assert not _oversize(launches)


# bf16, 384 columns: three 256 x 128 tiles per row block against two 256 x 256 ones
BF16_LONG = [(720000000, 8, 384), (720000000, 384, 8), ((1 << 31) - 4096, 8, 128), ((1 << 30) - 256, 8, 384)]


@pytest.mark.parametrize("T,di,do", BF16_LONG)
@pytest.mark.parametrize("r", [0, 8])
def test_bf16_launches_stay_within_a_dispatch(record, T, di, do, r):
    """The full waves of a two-launch product are of tiles that fit a dispatch, like the single launch."""
    for st, launches, _ in record([(c, T, di, do, r, "bf16", "cosnet", 1) for c in ("fwd", "bwd")]):
        assert st == 0 and launches
        assert not _oversize(launches)


def test_every_accepted_call_can_be_launched(record):
    """Shapes spread over the ABI's ranges: a call is refused before any launch, or all of its launches fit."""
    rng = random.Random(1)
    calls = []
    for _ in range(1500):
        G = rng.choice((1, 1, 2, 3, 4))
        T = min(int(2 ** rng.uniform(0, 31)), 2 ** 31 - 4096)
        di, do = (8 * max(1, int(2 ** rng.uniform(0, 17))) for _ in range(2))
        do = max(1, do // (8 * G)) * 8 * G
        dt = rng.choice(("bf16", "f32"))
        r = rng.choice((0, 8, 40, 128, 256 if dt == "bf16" else 96))
        act = rng.choice(("cosnet", "gelu", "cosnet3" if r <= 128 else "tanh_m"))
        calls += [(c, T, di, do, r, dt, act, G) for c in ("fwd", "bwd")]
    taken = 0
    for call, (st, launches, _) in zip(calls, record(calls)):
        assert not _oversize(launches), call
        assert st == 0 or not launches, call
        taken += st == 0
    assert taken > 2000


@pytest.mark.parametrize("act", ["cos", "gelu", "tanh", "leaky_relu"])
@pytest.mark.parametrize("G,r", [(1, 8), (1, 40), (3, 24), (1, 256)])
def test_unused_gradients_are_cleared_in_their_own_size(record, act, G, r):
    """One application: the given dM, domega2 and dphi2 are set to zero, dM in float32 (the public backward) or in the
    storage dtype (the binding's)."""
    size = {("bwd", "bf16"): 4, ("storage", "bf16"): 2, ("bwd", "f32"): 4, ("storage", "f32"): 4}
    calls = [(c, 300, 64, 8 * G, r, dt, act, G) for c, dt in size if dt == "bf16" or r <= 128]
    for call, (st, launches, zeros) in zip(calls, record(calls)):
        assert st == 0 and launches
        assert zeros["dM"] == G * r * r * size[call[0], call[5]], call
        assert zeros["domega2"] == zeros["dphi2"] == G * r * 4, call


def _tile(kernel):
    """"256x128" of a product kernel's name, None of any other kernel's."""
    m = re.search(r"gemm_tile_kernel<\w+, (\d+), (\d+), (\d+), (\d+),", kernel)
    if m:
        wm, wn, tm, tn = map(int, m.groups())
        return f"{32 * wm * tm}x{32 * wn * tn}"
    m = re.search(r"noble::gemm_kernel<float, (\d+), (\d+),", kernel)
    if m:
        return f"{m[1]}x{m[2]}"
    return "256x256" if "gemm_bf16_kernel" in kernel else "64x64" if "gemm_f32_kernel" in kernel else None


def _tiles(launches):
    return [t for t in (_tile(x[3]) for x in launches) if t]


@pytest.mark.parametrize("case", tiles.CASES, ids=[c[0] for c in tiles.CASES])
def test_tile_cases_run_their_tiles(record, case):
    name, T, di, do, r, G = case
    y, b = (_tiles(x[1]) for x in record([(c, T, di, do, r, "bf16", "cosnet", G) for c in ("fwd", "bwd")]))
    assert (y, b[:-1]) == tiles.TILES[name]   # the backward's last product: the weight gradients


@pytest.mark.parametrize("case", tiles.F32_CASES, ids=[c[0] for c in tiles.F32_CASES])
def test_float32_tile_cases_run_their_tiles(record, case):
    name, T, di, do, r, G = case
    y, b = (_tiles(x[1]) for x in record([(c, T, di, do, r, "f32", "cosnet", G) for c in ("fwd", "bwd")]))
    assert (*y, *b) == tiles.F32_TILES[name]


@pytest.mark.parametrize("case", split.CASES + split.CASES3, ids=[c[0] for c in split.CASES + split.CASES3])
def test_split_cases_run_their_forms(record, case):
    name, T, di, do, r, G = case
    three = case in split.CASES3
    tile, pieces, finish = (split.FORMS3 if three else split.FORMS)[name]
    act = "cosnet3" if three else "cosnet"
    full, static, least = record([
        ("fwd", T, di, do, r, "bf16", act, G), ("static", T, di, do, r, "bf16", act, G),
        ("fwd", T, di, do, r, "bf16", act, G, split._unsplit_scratch(T, di, do, r, G))])
    assert full == static   # the static scratch always holds the split form
    launches = full[1]
    assert _tiles(launches) == [tile]
    bm, bn = map(int, tile.split("x"))
    cdiv = lambda a, b: -(-a // b)
    assert launches[0][0] == pieces * cdiv(T, bm) * (cdiv(do, bn) + cdiv(G * r, bn))
    m = re.search(r"noble::(y_finish|chain_finish)_kernel(<\d>)?", launches[-1][3])
    assert m[1] + (m[2] or "") == finish
    assert len(launches) == (2 if finish == "chain_finish" else 3)
    assert "proj_kernel" in least[1][0][3]   # the least scratch: the unsplit form


def test_bench_names_the_kernel_it_reports(record):
    """The roofline entry's launch: the FFN-up projection's weight gradients, in the workgroups of the traffic record."""
    _, launches, _ = record([("bwd", 32768, 2048, 8192, 128, "bf16", "cosnet", 1)])[0]
    with open(bench.TRAFFIC_RECORD) as fh:
        rec = json.loads(re.search(r"^traffic_record: (\{.*\})$", fh.read(), re.M)[1])
    assert rec["kernel"] == bench.WGRAD_KERNEL
    assert [x[0] for x in launches if x[3].startswith(f"void {bench.WGRAD_KERNEL}(")] == [rec["workgroups"]]
