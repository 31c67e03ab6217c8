"""lb_column_stats and lb_mlp_forward at the sizes where their kernels change form.

Column statistics: one column, widths around the 256 columns of a block, row counts on both sides
of the change from one block per column to row runs with partial sums, ragged last runs.  Against
FP64 sums of the same data: the results are FP32 roundings of FP64 sums, so one FP32 ulp on the
mean's and the deviation's own scale.  Forward pass: sample counts around the 16 samples of a wave
and past one pass of the whole grid; each row's output must not depend on the rows beside it (bit
for bit), and pointers need only the alignment of a float.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dim", [(1, 1), (7, 3), (513, 255), (300, 256), (100, 257), (77, 1000), (20000, 36),
                                   (20001, 36), (50000, 15), (50001, 15), (60001, 1), (30011, 300), (200003, 36)])
def test_column_stats(lbrr, gpu, n, dim):
    torch = gpu
    g = torch.Generator(device="cuda")
    g.manual_seed(n + dim)
    x = torch.randn((n, dim), generator=g, device="cuda") * (1.0 + torch.arange(dim, device="cuda")) + 0.5
    mean, sd = torch.empty(dim, device="cuda"), torch.empty(dim, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    lbrr.check(lbrr.lb_column_stats(x.data_ptr(), n, dim, mean.data_ptr(), sd.data_ptr(), s))
    xd = x.double()
    ref = xd.std(0, unbiased=False)
    ref = torch.where(ref > 0, ref, torch.ones_like(ref))
    scale = xd.abs().mean(0) + ref
    assert ((mean.double() - xd.mean(0)).abs() <= 2.0**-23 * scale).all()
    assert ((sd.double() - ref).abs() <= 2.0**-23 * ref + 1e-12 * scale).all()
    m2, s2 = torch.empty_like(mean), torch.empty_like(sd)
    lbrr.check(lbrr.lb_column_stats(x.data_ptr(), n, dim, m2.data_ptr(), s2.data_ptr(), s))
    assert torch.equal(mean, m2) and torch.equal(sd, s2)


def test_column_stats_under_capture(lbrr, gpu):
    """Row runs need scratch, which a captured stream cannot allocate: the call still works there."""
    torch = gpu
    x = torch.randn((30000, 36), device="cuda")
    mean, sd = torch.empty(36, device="cuda"), torch.empty(36, device="cuda")
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        lbrr.check(lbrr.lb_column_stats(x.data_ptr(), 30000, 36, mean.data_ptr(), sd.data_ptr(), s.cuda_stream))
    for k in range(3):
        x.normal_(mean=float(k))
        g.replay()
        torch.cuda.synchronize()
        assert torch.allclose(mean.double(), x.double().mean(0), rtol=1e-6, atol=1e-7)
        assert torch.allclose(sd.double(), x.double().std(0, unbiased=False), rtol=1e-6)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, 2048 * 16 + 5])
def test_forward_rows_are_independent(lbrr, gpu, n):
    torch = gpu
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    buf = torch.randn(1 + 6723 + 78 + n * 36, generator=g, device="cuda")
    params, norm, x = 0.1 * buf[1:6724], buf[6724:6802].abs() + 0.5, buf[6802:]
    odd = torch.empty(6723 + 1, device="cuda")  # parameters at an address that is only 4-byte aligned
    odd[1:] = params
    s = torch.cuda.current_stream().cuda_stream
    y = torch.full((n + 1, 3), 7.0, device="cuda")
    lbrr.check(lbrr.lb_mlp_forward(odd[1:].data_ptr(), norm.data_ptr(), x.data_ptr(), n, y.data_ptr(), s))
    assert (y[n] == 7.0).all() and torch.isfinite(y).all()
    for k in {0, n // 2, n - 1}:
        one = torch.empty((1, 3), device="cuda")
        row = x[36 * k:36 * (k + 1)].contiguous()
        lbrr.check(lbrr.lb_mlp_forward(params.data_ptr(), norm.data_ptr(), row.data_ptr(), 1, one.data_ptr(), s))
        assert torch.equal(one[0], y[k])
