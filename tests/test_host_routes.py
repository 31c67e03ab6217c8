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
import ctypes, json, re, sys, time, types
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
    ("D3Q27", 6400, 6400, 1, "fp32", 1, False), ("D3Q19", 7500, 7500, 2, "fp32", 0, True),
    ("D3Q19", 8192, 8192, 1, "fp32", 0, False), ("D3Q19", 8192, 8192, 3, "fp32", 4, False),
    ("D3Q19", 23000, 23000, 2, "fp64", 0, True), ("D3Q19", 23552, 23552, 1, "fp64", 0, False),
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


# Tile heights the 3D moment step is built for, with their columns (mom_rows_option, tile.hpp)
HEIGHTS = {"mom_fp32": ((13, 64), (11, 64), (8, 64)), "mom_fp64": ((5, 64), (4, 64), (12, 32))}


def planned(storage, nx, ny, nz):
    """(rows, blocks) of the cheapest plan, every chunk count of every height tried."""
    up = lambda a, b: -(-a // b)
    best = None
    for rows, width in HEIGHTS[storage]:
        gx, gy, weight = up(nx, width), up(ny, rows), 9.5 if width == 32 else rows + 3
        for chunks in range(1, nz + 1):
            lz = up(nz, chunks)
            groups = up(gy * up(nz, lz), 8)
            cost = up(gx * groups, 32) * (lz + 2) * weight
            if best is None or cost < best[0]:
                best = cost, rows, gx * 8 * groups
    return list(best[1:])


MOMENT_BOXES = [(1, 1, 1), (24, 24, 330), (330, 24, 24), (64, 64, 64), (75, 131, 150), (301, 130, 65), (31, 3, 997),
                (200, 200, 200), (256, 256, 256), (130, 60, 40), (1000, 7, 91),
                (65, 131, 150), (36, 60, 40), (25, 67, 273), (200, 131, 150)]


@pytest.mark.parametrize("storage", sorted(HEIGHTS))
def test_moment_plans_are_the_cheapest(child, storage):
    """The plan of a moment step, searched in jumps, is the one that trying every chunk count finds."""
    got = child(f"""
out = []
for nx, ny, nz in {MOMENT_BOXES!r}:
    code, names = launches(lambda: P.lb_step(handle("D3Q27", nx, ny, nz, {storage!r}), 1))
    assert code == 0 and "k_mstep_t" in names[-1]
    fake.fake_grid.restype = ctypes.POINTER(ctypes.c_uint32)
    out.append([int(re.search("Li4E[fd]Li([0-9]+)E", names[-1])[1]), fake.fake_grid(len(names) - 1)[0]])
report(out)
""")
    assert got == [planned(storage, *box) for box in MOMENT_BOXES]


def test_narrow_tiles_where_wide_ones_stay_half_empty(child):
    """FP64 moment boxes a little over a multiple of 64 columns take the tiles of 32 columns."""
    boxes = [(65, 131, 150), (65, 130, 301), (75, 131, 150), (130, 131, 150), (200, 131, 150)]
    names = child(f"""
report([launches(lambda: P.lb_step(handle("D3Q27", nx, ny, nz, "mom_fp64", walls), 1))[1][-1]
        for walls in (0, 7) for nx, ny, nz in {boxes!r}])
""")
    assert all("Li4EdLi12E" in n for n in names), names


def test_planning_a_long_box_takes_no_time(child):
    """A plan is made by every lb_step call: far below a launch's own time, however many planes there are."""
    us = child("""
h = handle("D3Q27", 24, 24, 65535, "mom_fp32")
best = 1e9
for _ in range(20):
    t = time.perf_counter()
    P.check(P.lb_step(h, 1))
    best = min(best, time.perf_counter() - t)
    fake.fake_reset()
report(best * 1e6)
""")
    print(f"{us:.1f} us a call")
    assert us < 200


@pytest.mark.parametrize("lattice,storage,shape,walls,pairs", [
    # half-empty tiles whose first and last columns are walls
    ("D3Q27", "fp32", (75, 131, 150), 1, False), ("D3Q19", "fp32", (75, 131, 150), 7, False),
    ("D3Q19", "fp64", (75, 131, 150), 1, False), ("D3Q19", "fp64", (65, 130, 301), 7, False),
    ("D3Q27", "fp32", (65, 130, 301), 7, True), ("D3Q19", "fp64", (75, 300, 300), 1, True),
    ("D3Q27", "fp32", (75, 131, 150), 6, True), ("D3Q19", "fp64", (75, 131, 150), 0, True),
    ("D3Q19", "fp32", (100, 131, 150), 1, True), ("D3Q19", "fp64", (128, 128, 128), 7, True),
    # few rows, few columns, few planes
    ("D3Q27", "fp32", (500, 1, 1000), 0, False), ("D3Q27", "fp32", (500, 2, 1000), 0, False),
    ("D3Q27", "fp32", (500, 3, 1000), 0, True), ("D3Q27", "fp32", (500, 5, 1000), 6, True),
    ("D3Q27", "fp32", (400, 5, 400), 6, False), ("D3Q19", "fp32", (400, 3, 400), 0, False),
    ("D3Q19", "fp32", (128, 128, 8), 0, False), ("D3Q19", "fp32", (163, 235, 8), 0, True),
    ("D3Q27", "fp64", (163, 1, 235), 0, False), ("D3Q27", "fp64", (163, 3, 235), 0, True),
    ("D3Q27", "fp64", (16, 400, 400), 0, False), ("D3Q27", "fp64", (22, 240, 240), 0, True),
    ("D3Q19", "fp64", (22, 240, 240), 6, False), ("D3Q19", "fp64", (500, 1000, 1), 0, False),
    ("D3Q19", "fp32", (500, 1000, 3), 6, False), ("D3Q19", "fp32", (500, 1000, 8), 6, True),
    # torn lines out of cache
    ("D3Q27", "fp32", (7, 400, 400), 0, True), ("D3Q27", "fp32", (11, 400, 400), 6, True),
    ("D3Q27", "fp32", (16, 400, 400), 6, False), ("D3Q27", "fp32", (7, 240, 240), 0, False),
    # no such kernel: its registers spill
    ("D3Q27", "fp64", (256, 256, 256), 4, False), ("D3Q19", "fp64", (256, 256, 256), 4, True),
    # cubes
    ("D3Q27", "fp32", (64, 64, 64), 0, True), ("D3Q19", "fp32", (256, 256, 256), 0, True),
    ("D3Q27", "fp64", (64, 64, 64), 0, True), ("D3Q27", "fp32", (40, 40, 40), 0, False),
])
def test_pairs_in_3d(child, lattice, storage, shape, walls, pairs):
    """Pairs where their plan fills the chip enough to be faster than single steps."""
    code, names = child(f"report(launches(lambda: P.lb_step(handle({lattice!r}, *{shape!r}, {storage!r}, {walls}), 4)))")
    steps = [n for n in names if "k_step" in n]
    assert code == 0 and len(steps) == (2 if pairs else 4), names


@pytest.mark.parametrize("storage,nx,ny,rows", [
    # rows a block takes; 0: single steps
    ("fp32", 64, 64, 1), ("fp32", 256, 256, 1), ("fp64", 256, 256, 1), ("fp64", 288, 288, 2), ("fp32", 384, 384, 2),
    ("fp32", 2048, 2048, 6), ("fp32", 20, 256, 1), ("fp32", 20, 1000, 2), ("fp32", 20, 3000, 0), ("fp32", 64, 3000, 0),
    ("fp32", 64, 20000, 6), ("fp64", 64, 1000, 0), ("fp64", 20, 20000, 0), ("fp64", 130, 3000, 4), ("fp32", 100000, 1, 1),
])
def test_pairs_in_2d(child, storage, nx, ny, rows):
    """Rows a block of a 2D pair takes: few while there are few blocks; narrow boxes with many rows keep single steps."""
    code, names = child(f"""
code, names = launches(lambda: P.lb_step(handle("D2Q9", {nx}, {ny}, 1, {storage!r}), 4))
fake.fake_grid.restype = ctypes.POINTER(ctypes.c_uint32)
report([code, [[n, fake.fake_grid(i)[0]] for i, n in enumerate(names) if "k_step" in n]])
""")
    assert code == 0 and len(names) == (2 if rows else 4), names
    if rows:
        assert all("k_step_pair2" in n and g == -(-nx // 254) * -(-ny // rows) for n, g in names), names


@pytest.mark.parametrize("storage,side,check,steps,launched", [
    # launches of two steps and of one
    ("fp32", 192, 0, 6, (2, 2)), ("fp32", 320, 0, 6, (0, 6)), ("fp32", 320, 0, 8, (4, 0)), ("fp32", 320, 4, 10, (4, 2)),
    ("fp32", 320, 0, 10, (4, 2)), ("fp32", 320, 7, 27, (8, 11)), ("fp32", 320, 6, 7, (2, 3)), ("fp64", 256, 0, 5, (0, 5)),
    ("fp64", 256, 0, 7, (0, 7)), ("fp64", 256, 0, 4, (2, 0)), ("fp64", 256, 0, 12, (6, 0)), ("fp64", 512, 0, 7, (2, 3)),
    ("fp32", 512, 5, 13, (4, 5)), ("fp32", 64, 1, 9, (0, 9)), ("fp32", 64, 0, 3, (0, 3)),
])
def test_steps_left_over_by_pairs(child, storage, side, check, steps, launched):
    """Pairs two at a time up to the end of the call or the next check, then single steps; calls of five to seven
    steps stay single where the caches of the XCDs hold a 2D state."""
    code, names = child(f"""
h = handle("D2Q9", {side}, {side}, 1, {storage!r})
P.check(P.lb_set_check_interval(h, {check}))
code, names = launches(lambda: P.lb_step(h, {steps}))
assert P.lb_step_count(h) == {steps}
report([code, [n for n in names if "k_step" in n]])
""")
    two = sum("k_step_pair2" in n for n in names)
    assert code == 0 and (two, len(names) - two) == launched, names


@pytest.mark.parametrize("n,dim,direct", [(20000, 1000, True), (20001, 16, True), (36000, 16, True), (40000, 16, False),
                                          (27000, 36, True), (28000, 36, False), (20001, 100, False), (50000, 15, True),
                                          (50001, 1, False), (2**31, 1, False), (30000, 2**20, False)])
def test_column_stats_form(child, n, dim, direct):
    """One block a column while that is done before scratch would be allocated."""
    code, names = child(f"report(launches(lambda: P.lb_column_stats(4096, {n}, {dim}, 8192, 12288, None)))")
    assert code == 0
    assert len(names) == (1 if direct else 2) and ("k_column_stats" in names[0]) == direct, names
