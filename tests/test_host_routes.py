"""Which kernels the library launches, and that it launches them, without a GPU.

The host code of the built library runs in a child process against a HIP runtime that does nothing and
records launches (fake_hip.c), so boxes of any size and failing runtime calls cost nothing here.
"""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, sys, time, types
sys.modules["torch"] = types.ModuleType("torch")  # the binding imports it first, for its HIP runtime
sys.path.insert(0, {root!r})
fake = ctypes.CDLL({fake!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_kernel.restype = ctypes.c_char_p
import paper_1505_06900_amd as P

def handle(lattice, nx, ny, nz, storage, walls=0, order=4):
    h = P.lb_create(P.LATTICES[lattice], nx, ny, nz, 0.6, order)
    assert h, P.lb_last_error()
    P.check(P.lb_config(h, P.STORAGE[storage], 1.0))
    P.check(P.lb_set_walls(h, walls))
    P.check(P.lb_init_fields(h, 4096, 8192, 0, P.LB_F64, 1))
    return h

def launches(call):
    fake.fake_reset()
    code = call()
    return code, [fake.fake_kernel(i).decode() for i in range(fake.fake_launches())]

def report(x):
    print("REPORT" + json.dumps(x))
"""


@pytest.fixture(scope="module")
def child(lbrr, tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-Werror", "-o", lib, os.path.join(HERE, "fake_hip.c")],
                   check=True)

    def run(code, **env):
        r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, fake=lib) + code], capture_output=True,
                           text=True, timeout=120, env={**os.environ, **env})
        assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
        return json.loads(next(line[6:] for line in r.stdout.splitlines() if line.startswith("REPORT")))

    return run


@pytest.mark.parametrize("lattice,nx,ny,nz,storage,walls,pairs", [
    # a plane of one population (its rows q apart) on both sides of 4 GiB of lane offsets
    ("D3Q27", 6300, 6300, 2, "fp32", 0, True), ("D3Q27", 6400, 6400, 1, "fp32", 0, False),
    ("D3Q27", 6400, 6400, 1, "fp32", 1, False), ("D3Q19", 7500, 7500, 1, "fp32", 0, True),
    ("D3Q19", 8192, 8192, 1, "fp32", 0, False), ("D3Q19", 8192, 8192, 3, "fp32", 4, False),
    ("D3Q19", 23000, 23000, 1, "fp64", 0, True), ("D3Q19", 23552, 23552, 1, "fp64", 0, False),
    # a row of a 2D box; its unwalled single step has the same limit
    ("D2Q9", (1 << 29) - 1, 1, 1, "fp64", 1, True), ("D2Q9", 1 << 29, 1, 1, "fp64", 1, False),
    ("D2Q9", (1 << 30) - 1, 1, 1, "fp32", 1, True), ("D2Q9", 1 << 30, 1, 1, "fp32", 1, False),
])
def test_boxes_past_the_pairs_addressing_take_single_steps(child, lattice, nx, ny, nz, storage, walls, pairs):
    """Step pairs address a plane (2D: a row) with 32-bit lane offsets; boxes beyond keep the single steps."""
    code, names = child(f"report(launches(lambda: P.lb_step(handle({lattice!r}, {nx}, {ny}, {nz}, {storage!r}, {walls}), 4)))")
    assert code == 0
    steps = [n for n in names if "k_step" in n]
    assert len(steps) == (2 if pairs else 4), steps
    assert all(("k_step_pair" in n) == pairs for n in steps), steps


@pytest.mark.parametrize("fail", ["fake_fail_pool_create", "fake_fail_pool_malloc", "fake_capturing", None])
def test_column_stats_without_scratch(child, fail):
    """Where the device gives no scratch the statistics take the form that needs none."""
    code, names = child(f"""
if {fail!r}: ctypes.c_int.in_dll(fake, {fail!r}).value = 1
report(launches(lambda: P.lb_column_stats(4096, 1000000, 36, 8192, 12288, None)))
""")
    assert code == 0
    assert len(names) == (1 if fail else 2) and ("k_column_stats" in names[0]) == bool(fail), names
