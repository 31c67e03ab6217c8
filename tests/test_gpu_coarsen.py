"""lb_closure_coarsen where its blocks change form: narrow boxes (a thread each) and wider ones,
boxes as wide as a block and wider, box counts that leave a block partly empty, both input types.
Against the same averages in FP64: the sums run over F*F terms in another order, so each carries at
most F*F ulp of its terms' magnitudes, a division and two products a few more.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("factor,ncx,ncy", [(1, 1, 1), (1, 300, 3), (2, 129, 5), (3, 86, 7), (4, 64, 64), (5, 103, 2),
                                            (7, 37, 3), (8, 33, 3), (16, 17, 2), (64, 5, 2), (100, 3, 2), (128, 3, 2), (129, 3, 2), (255, 2, 2), (256, 2, 1),
                                            (257, 2, 2), (600, 1, 2)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_box_averages(lbrr, gpu, factor, ncx, ncy, dtype):
    torch = gpu
    from paper_1505_06900_amd import _lib

    F, nx, ny = factor, ncx * factor, ncy * factor
    g = torch.Generator(device="cuda")
    g.manual_seed(F + ncx)
    real = torch.float64 if dtype == "f64" else torch.float32
    rand = lambda k, s: s * torch.randn((k, ny, nx), generator=g, device="cuda", dtype=torch.float64)
    rho, u, pi = (1 + rand(1, 0.02)).to(real), rand(2, 0.05).to(real), rand(3, 1e-3).to(real)
    rc, uc, pc = (torch.full((k, ncy, ncx), float("nan"), device="cuda", dtype=torch.float64) for k in (1, 2, 3))
    alpha, beta = 0.7, -1.3
    lbrr.check(lbrr.lb_closure_coarsen(rho.data_ptr(), u.data_ptr(), pi.data_ptr(),
                                       _lib.LB_F64 if dtype == "f64" else _lib.LB_F32, nx, ny, F, alpha, beta,
                                       rc.data_ptr(), uc.data_ptr(), pc.data_ptr(),
                                       torch.cuda.current_stream().cuda_stream))
    r, v, p = rho.double(), u.double(), pi.double()
    box = lambda x: x.reshape(x.shape[0], ncy, F, ncx, F).mean((2, 4))
    ref_r = box(r)
    ref_u = box(r * v) / ref_r
    vv = torch.stack((v[0] * v[0], v[0] * v[1], v[1] * v[1]))
    uu = torch.stack((ref_u[0] * ref_u[0], ref_u[0] * ref_u[1], ref_u[1] * ref_u[1]))
    ref_p = alpha * box(p) + beta * (box(r * vv) - ref_r * uu)
    ulp = (F * F + 16) * 2.0**-52
    assert ((rc - ref_r).abs() <= ulp * box(r.abs())).all()
    assert ((uc - ref_u).abs() <= ulp * box((r * v).abs()) / ref_r + 2 * ulp * ref_u.abs()).all()
    scale = abs(alpha) * box(p.abs()) + abs(beta) * (box((r * vv).abs()) + ref_r * 4 * box(v.abs()).amax(0) ** 2)
    assert ((pc - ref_p).abs() <= 2 * ulp * scale).all()
