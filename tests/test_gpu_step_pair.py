"""Launches of two population steps against single steps, bit for bit.

lb_step may take steps two to a launch (FP64 and FP32 population storage, with or without walls;
D3Q27 FP64 with walls keeps single steps); the single steps are held to the oracle elsewhere.  Boxes at the edges of the launch's tiles: one
node, fewer rows or planes than a tile, rows of 64 +- 1 nodes, chunk lengths that leave one
plane over, both tile heights; every order.  LBRR_PAIR_LZ=0 gives the single steps.
"""
import pytest

pytestmark = pytest.mark.gpu

ROWS = {("D3Q27", "fp32"): (8, 9), ("D3Q19", "fp32"): (13, 9), ("D3Q27", "fp64"): (4, 3), ("D3Q19", "fp64"): (4, 3)}
SHAPES = [(1, 1, 1), (3, 2, 130), (7, 19, 65), (25, 37, 63), (20, 26, 64)]


def _run(lbrr, torch, lattice, shape, order, storage, calls, check=0, walls=(False,) * 3):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    rho = 1.0 + 0.01 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    u = 0.03 * torch.randn((lbrr.DIM[lattice],) + shape, generator=g, device="cuda", dtype=torch.float64)
    sim = lbrr.Simulation(lattice, shape, 0.62, order, storage=storage)
    sim.set_walls(*walls)
    sim.set_check_interval(check)
    sim.init_fields(rho, u)
    for n in calls:
        sim.step(n)
    out, steps = sim.get_populations(), sim.steps
    sim.close()
    return out, steps


@pytest.mark.parametrize("lattice,order", [("D3Q27", n) for n in (2, 3, 4, 5, 6)] + [("D3Q19", n) for n in (2, 3, 4)])
@pytest.mark.parametrize("storage", ["fp32", "fp64"])
def test_pairs_equal_single_steps(lbrr, gpu, lattice, order, storage, monkeypatch):
    for shape in SHAPES:
        monkeypatch.setenv("LBRR_PAIR_LZ", "0")
        want, steps = _run(lbrr, gpu, lattice, shape, order, storage, [9])
        assert steps == 9
        for rows in ROWS[lattice, storage]:
            for lz in (1, 6, 24):
                monkeypatch.setenv("LBRR_PAIR_LZ", str(lz))
                monkeypatch.setenv("LBRR_PAIR_ROWS", str(rows))
                got, steps = _run(lbrr, gpu, lattice, shape, order, storage, [9])
                assert steps == 9
                assert gpu.isfinite(got).all()
                assert gpu.equal(got, want), (shape, rows, lz)


@pytest.mark.parametrize("storage", ["fp32", "fp64"])
def test_own_choice_splits_and_checks(lbrr, gpu, storage, monkeypatch):
    """The library's own plan on a box it pairs: one call of 23 steps, calls of 1 to 8 steps, and
    calls with a check interval that ends inside a pair all give the same state."""
    shape = (40, 70, 100)
    want, _ = _run(lbrr, gpu, "D3Q27", shape, 4, storage, [1] * 23)
    for calls, check in (([23], 0), ([4, 5, 6, 8], 0), ([2, 3, 7, 11], 0), ([23], 5), ([9, 14], 1), ([23], 6)):
        got, steps = _run(lbrr, gpu, "D3Q27", shape, 4, storage, calls, check)
        assert steps == 23
        assert gpu.equal(got, want), (calls, check)


@pytest.mark.parametrize("lattice,order", [("D3Q27", 2), ("D3Q27", 4), ("D3Q27", 6), ("D3Q19", 3), ("D3Q19", 4)])
@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("walls", [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 1)])
def test_pairs_equal_single_steps_walls(lbrr, gpu, lattice, order, storage, walls, monkeypatch):
    """Wall nodes, edges and corners in both steps of a launch, in the tile and on its rim."""
    for shape in [(3, 3, 3), (7, 19, 65), (20, 14, 64)]:
        monkeypatch.setenv("LBRR_PAIR_LZ", "0")
        want, _ = _run(lbrr, gpu, lattice, shape, order, storage, [9], walls=walls)
        for rows in ROWS[lattice, storage]:
            for lz in (1, 5):
                monkeypatch.setenv("LBRR_PAIR_LZ", str(lz))
                monkeypatch.setenv("LBRR_PAIR_ROWS", str(rows))
                got, steps = _run(lbrr, gpu, lattice, shape, order, storage, [9], walls=walls)
                assert steps == 9
                assert gpu.isfinite(got).all()
                assert gpu.equal(got, want), (shape, rows, lz)


@pytest.mark.parametrize("order", [2, 3, 4])
@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("walls", [(False, False), (True, False), (False, True), (True, True)])
def test_pairs_equal_single_steps_2d(lbrr, gpu, order, storage, walls, monkeypatch):
    """Rows around the 254 columns of a block, one to several blocks, chunks that divide the rows or not."""
    for shape in [(1, 1, 1), (1, 3, 3), (1, 5, 254), (1, 20, 255), (1, 33, 600), (1, 4, 256)]:
        if (walls[0] and shape[2] < 3) or (walls[1] and shape[1] < 3):
            continue
        monkeypatch.setenv("LBRR_PAIR_LZ", "0")
        want, _ = _run(lbrr, gpu, "D2Q9", shape, order, storage, [9], walls=walls + (False,))
        for lz in (1, 2, 6, 24):
            monkeypatch.setenv("LBRR_PAIR_LZ", str(lz))
            got, steps = _run(lbrr, gpu, "D2Q9", shape, order, storage, [9], walls=walls + (False,))
            assert steps == 9
            assert gpu.isfinite(got).all()
            assert gpu.equal(got, want), (shape, lz)


@pytest.mark.parametrize("lattice,shape,storage,walls", [
    ("D3Q27", (20, 26, 70), "fp32", (0, 0, 0)), ("D3Q19", (20, 26, 70), "fp64", (0, 0, 0)),
    ("D3Q19", (20, 26, 70), "fp32", (1, 1, 1)), ("D2Q9", (1, 33, 600), "fp64", (0, 1, 0))])
@pytest.mark.parametrize("steps", [8, 10])
def test_pairs_in_a_graph(lbrr, gpu, lattice, shape, storage, walls, steps, monkeypatch):
    """Captured launches of two steps, replayed between eager steps of the same handle and checked against the
    single steps of another after every replay.  10 steps: four pairs and two single steps."""
    torch = gpu
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    rho = 1.0 + 0.01 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    u = 0.03 * torch.randn((lbrr.DIM[lattice],) + shape, generator=g, device="cuda", dtype=torch.float64)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    sims = []
    with torch.cuda.stream(s):
        for _ in range(2):
            sim = lbrr.Simulation(lattice, shape, 0.62, 4, storage=storage, stream=s)
            sim.set_walls(*(bool(w) for w in walls))
            sims.append(sim.init_fields(rho, u))
    torch.cuda.synchronize()
    single, graphed = sims
    graph = torch.cuda.CUDAGraph()
    monkeypatch.setenv("LBRR_PAIR_LZ", "6")
    with torch.cuda.graph(graph, stream=s):
        graphed.step(steps)
    for k in range(4):
        with torch.cuda.stream(s):
            graph.replay()
            monkeypatch.setenv("LBRR_PAIR_LZ", "0")
            single.step(steps + 4)
            monkeypatch.setenv("LBRR_PAIR_LZ", "6")
            graphed.step(4)
        torch.cuda.synchronize()
        a, b = single.get_populations(), graphed.get_populations()
        torch.cuda.synchronize()
        assert torch.isfinite(a).all()
        assert torch.equal(a, b), f"replay {k + 1}"
    del graph
    for sim in sims:
        sim.close()
