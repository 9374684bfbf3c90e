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


def _with_fake_hip(tmp_path, program):
    """Run a Python program with the library on top of the stand-in for the HIP
    runtime (no GPU, no torch): `abi` and `fake` are there; returns what it
    printed last, as JSON."""
    lib = _compile("fake_hip.hip", tmp_path / "fake_hip.so")
    head = ("import ctypes as C, json, sys\n"
            "fake = C.CDLL(%r, mode=C.RTLD_GLOBAL)\n"
            "fake.fake_launches.restype = C.c_char_p\n"
            "fake.fake_steps.restype = C.c_int64\n"
            "sys.path.insert(0, %r)\n"
            "from paper_1312_1789_amd import abi\n"
            "assert 'torch' not in sys.modules\n" % (lib, build_lib.ROOT))
    r = subprocess.run([sys.executable, "-c", head + program], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.splitlines()[-1])


LARGE_CALLS = """
n = 1 << 26
cfg = abi.nbody_config(4, abi.NBODY_MIXED, n, 0, 1e-8, 0.01, 0.01, 3, 20, 0, 0.0, 0)
at = 1 << 40   # device addresses, never read here
ctx = abi.nbody_create(cfg, at, abi.nbody_workspace_size(cfg), 0)
st = abi.nbody_state(at, at, at, (C.c_void_p * 6)(at, at), at, at)
seen = []
for fuse in (1, 0):
    abi.nbody_set_fusion(ctx, fuse)
    for n_split in (0, 1, 8):
        abi.nbody_set_launch(ctx, 1, 64, n_split, 3)
        for n_act in (64 * 65535, 64 * 65535 + 1, n):
            fake.fake_launches()
            abi.nbody_predict_force(ctx, st, 1, n_act, at, at, at, 0, 0, at)
            rows = [l.split() for l in fake.fake_launches().decode().splitlines()]
            seen += [(fuse, n_act, l[0], *map(int, l[1:])) for l in rows if "force" in l[0]]
print(json.dumps(seen))
"""


def test_wave_split_launches_within_limits(tmp_path):
    """The wave j-split kernels, with the predictor inside and without, take
    every active set a context can have (a shape set by hand is used for any
    number of rows): more than 65535 tiles of 64 rows do not fit the second
    grid dimension."""
    seen = _with_fake_hip(tmp_path, LARGE_CALLS)
    assert len(seen) == 18
    for fuse, n_act, name, gx, gy, gz, bx in seen:
        rows = 64 if fuse else 16
        assert ("small" in name) == (fuse == 1)
        assert gx * rows >= n_act and gy <= 65535 and gz == 1, (name, n_act, gx, gy)


FAILED_LAUNCHES = """
n = 1024
cfg = abi.nbody_config(4, abi.NBODY_FP64, n, 0, 1e-8, 0.01, 0.01, 3, 20, 0, 0.0, 0)
size = abi.nbody_workspace_size(cfg)
import numpy as np
ws = np.zeros(size + 256, np.uint8)   # "device" memory, which the stand-in's step kernel writes
at = (ws.ctypes.data + 255) // 256 * 256
ctx = abi.nbody_create(cfg, at, size, 0)
st = abi.nbody_state(at, at, at, (C.c_void_p * 6)(at, at), at, at)
lib, seen = abi.lib(), []
def run(max_steps):
    steps, t = C.c_int64(-1), C.c_int64(-1)
    before = fake.fake_steps()
    rc = lib.nbody_run(ctx, C.byref(st), C.c_int64(1 << 60), C.c_int64(max_steps), C.byref(steps), C.byref(t))
    s = abi.nbody_get_stats(ctx)
    return [rc, steps.value, t.value, fake.fake_steps() - before, fake.fake_steps(), fake.fake_queued(), s.steps]
for n_act in (1, 700):      # steps enqueued ahead, and steps sized by the host
    for fail_at in range(1, 26):
        fake.fake_script(C.c_int64(n_act), fail_at)
        seen.append(run(5))
        fake.fake_script(C.c_int64(n_act), 0)
        seen.append(run(3))
print(json.dumps(seen))
"""


def test_steps_after_a_failed_launch(tmp_path):
    """A launch of a run that fails, each in turn: the call reports the error and
    the steps that were taken, steps enqueued ahead included, with nothing left in
    flight; the next run starts from a schedule of its own, not from one that
    a step enqueued ahead published for the run before."""
    seen = _with_fake_hip(tmp_path, FAILED_LAUNCHES)
    failed = [s for s in seen if s[0] != 0]
    assert len(failed) >= 20 and all(s[0] == -2 for s in failed)
    for rc, steps, t, taken, total, queued, counted in seen:
        assert (steps, counted, queued) == (taken, total, 0)
        assert t == (total if steps else 0)
        if rc == 0:
            assert steps in (3, 5)
    assert any(0 < s[1] < 5 for s in failed)
