"""Instance normalisation of small volumes (statistics and backward pass in one launch each) against fp64, where its
parts can go wrong: fewer voxels than lanes, volumes that end inside a wave and inside a thread's pieces, the last
volume of each form and the first of the next, channel counts whose lines of 128 bytes are cut by a sample's end, and
work items that do not divide by the XCDs."""
import pytest
import torch

from paper_1812_07816_amd import glue

pytestmark = pytest.mark.gpu

SLOPE, EPS = 0.01, 1e-5


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("N,V,C", [(1, 1, 8), (3, 2, 40), (2, 63, 512), (1, 64, 24), (2, 65, 72), (1, 1023, 8), (2, 1024, 32), (3, 1025, 40),
                                   (1, 2048, 64), (1, 2049, 16), (1, 3300, 320), (2, 4096, 72),
                                   (1, 1536, 24), (1, 1537, 24), (4, 2048, 64), (2, 2560, 16), (2, 2561, 16), (8, 4096, 64), (32, 2600, 312)])
def test_small_volumes_match_fp64(device, dtype, N, V, C):
    gen = torch.Generator(device="cuda").manual_seed(V + C)
    rnd = lambda: torch.randn((N, V, 1, 1, C), generator=gen, device="cuda")
    z, da = (2 * rnd() + 3 * rnd()[:, :1]).to(dtype), rnd().to(dtype)     # (a channel's mean of several standard deviations)
    ws = glue.instnorm_workspace(N, C)
    guard = torch.full((N * C + 64, 2), 7.0, device="cuda")
    stats = guard[:N * C].view(N, C, 2)
    glue.instnorm_stats(z, stats, ws)
    z64 = z.double()
    mean, var = z64.mean((1, 2, 3)), z64.var((1, 2, 3), unbiased=False)
    # sums in fp64: the results carry one rounding to fp32; the variance is a difference of squares, each within 2^-52 V
    assert bool(((stats[..., 0].double() - mean).abs() <= 2.0 ** -23 * mean.abs() + 1e-30).all())
    rel = 2.0 ** -23 + 2.0 ** -52 * (V + 8) * (1 + mean.square() / (var + EPS))
    rstd = (var + EPS).rsqrt()
    assert bool(((stats[..., 1].double() - rstd).abs() <= rel * rstd).all())
    assert bool((guard[N * C:] == 7).all())

    a = z.clone()
    glue.instnorm_lrelu_fwd(a, stats, SLOPE)
    got = da.clone()
    glue.instnorm_lrelu_bwd(got, a, stats, ws, SLOPE)
    a64, g64 = a.double(), da.double()
    gg, xh = torch.where(a64 > 0, g64, SLOPE * g64), torch.where(a64 > 0, a64, a64 / SLOPE)
    m1, m2 = gg.mean((1, 2, 3), keepdim=True), (gg * xh).mean((1, 2, 3), keepdim=True)
    r = stats[..., 1].double().view(N, 1, 1, 1, C)
    ref = r * (gg - m1 - xh * m2)
    # the terms in fp32 (the slope and its inverse too): eight roundings of at most 2^-24 each; m1 and m2 are sums of such
    # terms; the result is rounded once to its type
    size = r * (gg.abs() + gg.abs().mean((1, 2, 3), keepdim=True) + xh.abs() * (gg * xh).abs().mean((1, 2, 3), keepdim=True))
    tol = 8 * 2.0 ** -24 * size + (2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23) * ref.abs()
    assert bool(((got.double() - ref).abs() <= tol + 1e-30).all())
    again = da.clone()
    glue.instnorm_lrelu_bwd(again, a, stats, ws, SLOPE)
    assert torch.equal(got, again)
