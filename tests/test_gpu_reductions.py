"""lb_reduce and lb_enstrophy at the sizes where their launches change form.

One block per 256 nodes; up to 256 blocks the last one to finish adds the partial sums, beyond that
a launch of its own does.  Grids on both sides of both lines, called repeatedly (each call must find
the blocks' ticket as the first did) and from many handles (more than there are pinned result
slots), against FP64 sums of the fields: both sides are FP64 sums of the same values in different
orders, so 1e-13 of the sum of magnitudes.
"""
import pytest

pytestmark = pytest.mark.gpu


def _sim(lbrr, torch, lattice, shape, storage):
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(shape))
    d = lbrr.DIM[lattice]
    rho = 1.0 + 0.01 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    u = 0.02 + 0.03 * torch.randn((d,) + shape, generator=g, device="cuda", dtype=torch.float64)
    return lbrr.Simulation(lattice, shape, 0.6, 4, storage=storage).init_fields(rho, u)


def _enstrophy(torch, u):
    dd = lambda a, dim: 0.5 * (torch.roll(a, -1, dim) - torch.roll(a, 1, dim))
    if len(u) == 2:
        w2 = (dd(u[1], 2) - dd(u[0], 1)) ** 2
    else:
        w2 = ((dd(u[2], 1) - dd(u[1], 0)) ** 2 + (dd(u[0], 0) - dd(u[2], 2)) ** 2 + (dd(u[1], 2) - dd(u[0], 1)) ** 2)
    return float(0.5 * w2.mean())


@pytest.mark.parametrize("storage", ["fp64", "mom_fp64"])
@pytest.mark.parametrize("lattice,shape", [("D2Q9", (1, 1, 1)), ("D2Q9", (1, 5, 51)), ("D2Q9", (1, 16, 16)),
                                           ("D2Q9", (1, 1, 257)), ("D2Q9", (1, 256, 256)), ("D2Q9", (1, 1, 65537)),
                                           ("D3Q19", (16, 64, 64)), ("D3Q27", (17, 64, 61)), ("D3Q27", (65, 100, 90))])
def test_totals_and_enstrophy(lbrr, gpu, lattice, shape, storage):
    torch = gpu
    sim = _sim(lbrr, torch, lattice, shape, storage)
    rho, u = sim.moments()
    want = [float(rho.sum())] + [float((rho * c).sum()) for c in u] + [0.0] * (3 - len(u))
    want.append(float(0.5 * (rho * (u * u).sum(0)).sum()))
    scale = [float(rho.sum())] + [float((rho * c).abs().sum()) for c in u] + [1.0] * (3 - len(u)) + [want[4]]
    first = sim.reduce()
    for got, ref, s in zip(first, want, scale):
        assert abs(got - ref) <= 1e-13 * s
    e = sim.enstrophy()
    assert e == pytest.approx(_enstrophy(torch, u), rel=1e-12, abs=1e-18)
    for _ in range(5):
        assert sim.reduce() == first
        assert sim.enstrophy() == e
    sim.close()


def test_more_handles_than_result_slots(lbrr, gpu):
    sims = [_sim(lbrr, gpu, "D2Q9", (1, 4, 4 + k % 3), "fp64") for k in range(300)]
    got = [s.reduce() for s in sims]
    assert all(got[k] == got[k % 3] for k in range(300)) and got[0] != got[1]
    for s in sims[::2]:
        s.close()
    again = _sim(lbrr, gpu, "D2Q9", (1, 4, 4), "fp64")
    assert again.reduce() == got[0]
    for s in sims[1::2] + [again]:
        s.close()
