"""Host parts of the library and code that both sides compile, on the CPU."""
import json
import os
import subprocess
import sys

import numpy as np

from paper_1312_1789_amd import build_lib

NATIVE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native")
MAX_ROWS = 1 << 22   # kBatchMaxRows


def _compile(name, out):
    """tests/native/<name> as a shared library of host code."""
    subprocess.run([build_lib.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-x", "hip",
                    "-I", os.path.join(build_lib.ROOT, "include"), "-I", build_lib.CSRC,
                    os.path.join(NATIVE, name), "-o", str(out)], check=True)
    return str(out)


PLAN_CALL = """
import ctypes as C, json, sys
import numpy as np
f = C.CDLL(sys.argv[1]).batch_plan
f.argtypes = [C.c_int, C.c_void_p, C.c_void_p] + [C.c_int] * 5 + [C.c_void_p]
for line in sys.stdin:
    nn, na, shape = json.loads(line)
    nn, na, out = np.array(nn, np.int64), np.array(na, np.int64), np.zeros(4, np.int64)
    f(len(nn), nn.ctypes.data, na.ctypes.data, *shape, out.ctypes.data)
    print(json.dumps(out.tolist()), flush=True)
"""


def test_batch_plan_cuts(tmp_path):
    """Every launch shape the batched form accepts, from one workgroup on, over
    steps from all clusters resting to all particles active: the plan divides
    by no zero (that would end the process it runs in), and its partial rows
    stay within the scratch, i_tile x items aimed for + n."""
    lib = _compile("batch_plan.hip", tmp_path / "batch_plan.so")
    rng = np.random.default_rng(61)
    cases = []
    for grid in (1, 2, 7, 8, 9, 64, 1024, 3072, 1 << 20):
        for per_wg, itile, halves, grain in ((1, 64, 2, 64), (8, 64, 1, 128), (32, 128, 1, 64), (8, 256, 1, 128)):
            for nc, top in ((1, 40), (5, 100), (40, 3000), (300, 60), (2, 200000)):
                nn = rng.integers(1, top + 1, nc)
                for na in (0 * nn, np.minimum(nn, 1), nn * (rng.random(nc) < 0.3), rng.integers(0, nn + 1), nn):
                    cases.append((nn.tolist(), na.tolist(), (grid, per_wg, itile, halves, grain)))
    r = subprocess.run([sys.executable, "-c", PLAN_CALL, lib], input="\n".join(json.dumps(c) for c in cases),
                       capture_output=True, text=True)
    got = [json.loads(x) for x in r.stdout.splitlines()]
    assert r.returncode == 0 and len(got) == len(cases), (r.returncode, cases[min(len(got), len(cases) - 1)])
    for (nn, na, shape), (items, rows, least, most) in zip(cases, got):
        grid, per_wg, itile = shape[:3]
        assert rows <= min(grid * per_wg * itile, MAX_ROWS) + sum(nn), (nn, na, shape)
        if sum(na) == 0:
            assert items == 0
        else:
            assert 1 <= least <= most
        if grid == 1 and sum((a + itile - 1) // itile * itile * n for n, a in zip(nn, na)) < 4 * 32768:
            assert sum(na) == 0 or most == 1   # one workgroup, little work: nothing is split
