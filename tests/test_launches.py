"""The launches of libnoble's calls, recorded on the CPU by
tests/c/launch_record.cpp (HIP's launch function replaced, no GPU): what the
launch rules choose, and that every launch can be made."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2603_06492_amd import noble

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
