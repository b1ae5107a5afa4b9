"""Errors of the fp32 layers against 64 bits, next to those of the fp32 matrix instructions on the same operands: products from
bf16 parts (implicit GEMM, weight gradient over numbered positions) and the kernels of the smallest layers are no further from
the exact sums."""
import pytest
import torch

from paper_1812_07816_amd import conv3d as mc

pytestmark = pytest.mark.gpu

# (N, D, H, W, Cin, Cout, k, s, p) and the relative errors (2-norm) of forward pass, data gradient and weight gradient on the
# operands below by the kernels that served these layers before: f32_gconv_kernel (data gradients with 32 and more channels in
# strided layers, and layers of 256 and more: f32s_gconv_kernel) and f32_wgrad_kernel or, up to 4 channels, f32_wgrad_c4_kernel
LAYERS = [
    ((1, 24, 24, 24, 64, 128, 2, 2, 0), (4.043e-07, 2.039e-07, 1.943e-07)),
    ((2, 20, 22, 18, 32, 64, 3, 2, 1), (5.077e-07, 2.453e-07, 1.669e-07)),
    ((1, 15, 16, 17, 128, 256, 3, 2, 1), (9.812e-07, 5.083e-07, 1.511e-07)),
    ((2, 8, 8, 8, 320, 320, 3, 1, 1), (1.351e-06, 1.348e-06, 2.582e-07)),
    ((1, 10, 12, 11, 256, 64, 3, 1, 1), (1.229e-06, 6.016e-07, 2.722e-07)),
    ((2, 19, 18, 21, 20, 44, 3, 2, 0), (4.149e-07, 2.397e-07, 1.791e-07)),
    ((1, 12, 14, 13, 40, 72, 3, 1, 2), (5.263e-07, 7.941e-07, 2.934e-07)),
    ((1, 16, 16, 16, 4, 8, 3, 1, 1), (1.758e-07, 2.505e-07, 2.054e-07)),
    ((2, 9, 8, 7, 8, 16, 3, 1, 1), (2.386e-07, 2.734e-07, 2.583e-07)),
    ((1, 6, 9, 8, 5, 7, 3, 1, 1), (1.872e-07, 2.258e-07, 1.969e-07)),
    ((1, 12, 11, 11, 3, 32, 3, 1, 1), (1.529e-07, 4.098e-07, 1.701e-07)),
    ((1, 13, 16, 13, 5, 12, 3, 1, 1), (1.980e-07, 3.015e-07, 3.138e-07)),
]


def operands(case):
    N, D, H, W, Cin, Cout, k, s, p = case
    gen = torch.Generator().manual_seed(sum(case))
    o = [(v + 2 * p - k) // s + 1 for v in (D, H, W)]
    rnd = lambda *shape: torch.randn(shape, generator=gen)
    return rnd(N, D, H, W, Cin), rnd(Cout, k, k, k, Cin) * (2 / (k ** 3 * Cin)) ** 0.5, rnd(N, *o, Cout)


def errors(case):
    N, D, H, W, Cin, Cout, k, s, p = case
    x, w, dy = operands(case)
    d = mc.make_desc(*case, torch.float32)
    first = lambda t: t.double().permute(0, 4, 1, 2, 3).contiguous()
    last = lambda t: t.permute(0, 2, 3, 4, 1)
    X, Wt, DY = first(x), first(w), first(dy)
    refs = (last(torch.nn.functional.conv3d(X, Wt, stride=s, padding=p)), last(torch.nn.grad.conv3d_input(X.shape, Wt, DY, stride=s, padding=p)),
            last(torch.nn.grad.conv3d_weight(X, Wt.shape, DY, stride=s, padding=p)))
    xd, wd, dyd = x.cuda(), w.cuda(), dy.cuda()
    got = mc.conv3d_fwd(d, xd, wd), mc.conv3d_dgrad(d, dyd, wd), mc.conv3d_wgrad(d, xd, dyd)
    return [float((g.cpu().double() - r).norm() / r.norm()) for g, r in zip(got, refs)]


@pytest.mark.parametrize("case, former", LAYERS, ids=["x".join(map(str, c[:4])) + "-" + "-".join(map(str, c[4:])) for c, _ in LAYERS])
def test_errors_are_no_larger_than_those_of_the_fp32_instructions(device, case, former):
    d = mc.make_desc(*case, torch.float32)
    got = errors(case)
    print(case, [f"{e:.2e}" for e in got], [mc.kernel_detail(d, q) for q in range(3)], flush=True)
    for e, f in zip(got, former):
        assert e <= f, (case, got, former)
