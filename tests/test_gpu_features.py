"""lb_closure_features at the edges of its 64 x 4 tiles: grids of one node, narrower than the stencil's
wrap, one past a tile, and every population storage.  Against the moments of the same state: both are
formed from nine populations of size below 1 in 32 bits at least, so within 64 ulp of 1.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx", [(1, 1), (2, 3), (3, 2), (4, 64), (5, 65), (9, 130), (1, 200), (70, 1)])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16"])
def test_features(lbrr, gpu, ny, nx, storage):
    torch = gpu
    import paper_1505_06900_amd as P

    g = torch.Generator(device="cuda")
    g.manual_seed(nx * 100 + ny)
    shape = (1, ny, nx)
    rand = lambda k, s: s * torch.randn((k,) + shape, generator=g, device="cuda", dtype=torch.float64)
    sim = P.Simulation("D2Q9", shape, 0.6, 4, storage=storage)
    sim.init_fields(1 + rand(1, 0.02)[0], rand(2, 0.05), rand(3, 1e-3))
    feat, lab = sim.closure_features(a_target=None, plain_weight=0.0)
    rho, u = sim.moments()[:2]
    sim.close()
    m = torch.stack((rho.reshape(ny, nx) - 1, *u.reshape(2, ny, nx))).double()
    assert (lab == 0).all()
    feat = feat.reshape(ny, nx, 36).double()
    bar = 64 * 2.0**-24
    for dy in range(3):
        for dx in range(3):
            near = torch.roll(m, (1 - dy, 1 - dx), (1, 2)).permute(1, 2, 0)
            got = feat[..., 9 + 3 * (3 * dy + dx): 12 + 3 * (3 * dy + dx)]
            assert (got - near).abs().max() <= bar, (dy, dx)
    # the pulled deviations of all nodes are the stored ones, moved: equal sums
    assert (feat[..., :9].sum((0, 1, 2)) - m[0].sum()).abs() <= nx * ny * bar
