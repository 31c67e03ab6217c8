"""The 32-column tiles of the FP64 moment step: boxes around 32 columns and 12 rows, periodic and walled.
Tile height and width do not enter the arithmetic, so the state has the bits of the 64-column tiles'.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 3, 3), (7, 12, 32), (9, 13, 31), (20, 25, 25), (5, 24, 1), (6, 40, 33)])
@pytest.mark.parametrize("lattice,order", [("D3Q19", 4), ("D3Q27", 6)])
@pytest.mark.parametrize("walls", [(False, False, False), (True, True, True)])
def test_same_bits(lbrr, gpu, monkeypatch, shape, lattice, order, walls):
    torch = gpu
    import paper_1505_06900_amd as P

    if any(walls) and min(shape) < 2:
        pytest.skip("a walled axis needs two nodes")
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(shape))
    rho = 1 + 0.01 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    u = 0.03 * torch.randn((3,) + shape, generator=g, device="cuda", dtype=torch.float64)
    out = {}
    for rows in ("12", "5"):
        monkeypatch.setenv("LBRR_MOM_ROWS", rows)
        sim = P.Simulation(lattice, shape, 0.62, order, storage="mom_fp64")
        sim.set_walls(*walls)
        sim.init_fields(rho, u)
        sim.step(5)
        out[rows] = sim.moments(pi1=True)
        sim.close()
    assert all(torch.isfinite(x).all() for x in out["5"])
    assert all(torch.equal(x, y) for x, y in zip(out["12"], out["5"]))


@pytest.mark.parametrize("storage,rows", [("mom_fp32", (13, 11, 8)), ("mom_fp64", (12, 5, 4))])
@pytest.mark.parametrize("lattice,order", [("D3Q19", 4), ("D3Q27", 4), ("D3Q27", 6)])
@pytest.mark.parametrize("walls", [(False, False, False), (True, True, True), (False, True, False)])
def test_every_tile_height(lbrr, gpu, monkeypatch, storage, rows, lattice, order, walls):
    """Each height the 3D moment step is built for, on boxes around its rows and 64 columns, with chunks of one
    plane, odd, even and ragged ones: one set of bits, and the oracle's fields (test_gpu_walls.py's bars)."""
    import numpy as np
    import test_gpu_parity as TP
    import test_gpu_walls as TW

    tol = TW.TOL[storage]
    for shape in [(7, 11, 63), (6, 14, 65), (5, 26, 129)]:
        ref = TW.oracle_walls(lattice, order, 0.63, shape, walls, 5, 17)
        first = None
        for height in rows:
            for lz in ("1", "3", "4", "64"):
                monkeypatch.setenv("LBRR_MOM_ROWS", str(height))
                monkeypatch.setenv("LBRR_MOM_LZ", lz)
                got = TW.gpu_walls(lbrr, lattice, order, 0.63, shape, walls, 5, 17, storage)
                if first is None:
                    first = got
                    e = [max(TP.rel_l2(g, r), TP.rel_linf(g, r)) for g, r in zip(got[:3], ref[:3])]
                    assert e[0] <= tol[0] and e[1] <= tol[0] and e[2] <= tol[1], (shape, e)
                assert all(np.array_equal(a, b) for a, b in zip(got[:3], first[:3])), (shape, height, lz)
