"""The smallest fp32 layers (one launch a pass) against the fp64 oracle, where the kernels can go wrong: channels one and
four at a time, output channels that end inside a group of eight, fewer positions than lanes, positions that end inside a
wave, strides that skip voxels, taps that miss the volume on both sides, and every fused epilogue."""
import numpy as np
import pytest
import torch

from paper_1812_07816_amd import conv3d as mc
from oracle import conv3d as oc
from tests import parity

pytestmark = pytest.mark.gpu

# sums of n <= 8192 fp32 products: n * 2^-24 of sum |a b| at the very worst; measured 3e-7 of max(|ref|, rms)
TOL = 4e-6

CASES = [
    # N, D, H, W, Cin, Cout, k, s, p, passes
    ((1, 1, 1, 1, 1, 1, 3, 1, 1), "012"),
    ((1, 16, 16, 16, 4, 8, 3, 1, 1), "012"),
    ((2, 3, 5, 7, 3, 5, 3, 1, 1), "012"),
    ((1, 9, 10, 11, 2, 32, 3, 1, 1), "012"),
    ((2, 7, 6, 9, 8, 20, 3, 2, 1), "012"),
    ((1, 8, 9, 10, 12, 28, 3, 2, 0), "012"),
    ((3, 5, 4, 7, 6, 9, 2, 2, 0), "012"),      # voxels no tap reaches
    ((1, 6, 5, 4, 20, 16, 3, 1, 2), "012"),    # outputs larger than the input
    ((2, 5, 5, 5, 8, 200, 1, 1, 0), "012"),
    ((1, 2, 31, 1, 32, 4, 3, 1, 1), "012"),
    ((2, 16, 16, 16, 4, 12, 3, 1, 1), "012"),  # the most positions of a weight gradient
    ((1, 15, 16, 17, 5, 8, 3, 1, 1), "012"),
]


@pytest.mark.parametrize("case, passes", CASES, ids=["x".join(map(str, c[:4])) + "-" + "-".join(map(str, c[4:])) for c, _ in CASES])
def test_matches_oracle(device, case, passes):
    d = mc.make_desc(*case, torch.float32)
    assert "".join(str(q) for q in range(3) if mc.kernel_detail(d, q) == "f32_direct") == passes
    errs = parity.run_case(98, 800 + CASES.index((case, passes)), *case, bf16=False, full=True)
    assert max(errs.values()) <= TOL, errs


@pytest.mark.parametrize("k, s, p", [((1, 2, 2), (1, 2, 2), 0), ((3, 3, 3), (1, 2, 2), 1), ((2, 3, 1), (2, 1, 1), (0, 1, 0)), ((3, 1, 2), (1, 1, 2), (1, 0, 0))])
def test_axes_of_their_own(device, k, s, p):
    g = torch.Generator().manual_seed(4)
    x, w = torch.randn((2, 6, 6, 9, 10), generator=g).double(), torch.randn((12, 6, *k), generator=g).double()
    d = mc.make_desc(2, 6, 9, 10, 6, 12, k, s, p, torch.float32)
    assert all(mc.kernel_detail(d, q) == "f32_direct" for q in range(3))
    y = torch.nn.functional.conv3d(x, w, stride=s, padding=p)
    dy = torch.randn(y.shape, generator=g).double()
    dx = torch.nn.grad.conv3d_input(x.shape, w, dy, stride=s, padding=p)
    dw = torch.nn.grad.conv3d_weight(x, w.shape, dy, stride=s, padding=p)
    dev = lambda t: t.permute(0, 2, 3, 4, 1).float().contiguous().cuda()
    for got, ref in ((mc.conv3d_fwd(d, dev(x), dev(w)), y), (mc.conv3d_dgrad(d, dev(dy), dev(w)), dx), (mc.conv3d_wgrad(d, dev(x), dev(dy)), dw)):
        e = got.cpu().double().permute(0, 4, 1, 2, 3) - ref
        assert float(e.abs().max() / ref.square().mean().sqrt()) <= TOL


@pytest.mark.parametrize("case", [(1, 6, 7, 5, 4, 8, 3, 1, 1), (2, 6, 8, 6, 6, 10, 3, 2, 1)])
def test_epilogues_and_values_that_must_not_spread(device, case):
    d = mc.make_desc(*case, torch.float32)
    xs, wsh, ys = mc._shapes(d)
    torch.manual_seed(2)
    x, w, dy, add, ref = (torch.randn(v, device="cuda") for v in (xs, wsh, ys, xs, xs))
    y, dx = mc.conv3d_fwd(d, x, w), mc.conv3d_dgrad(d, dy, w)
    assert torch.equal(mc.conv3d_fwd_lrelu(d, x, w, 0.01), torch.where(y > 0, y, 0.01 * y))
    f = torch.where(ref > 0, 1.0, 0.01)
    assert torch.equal(mc.conv3d_dgrad_lrelu(d, dy, w, ref, 0.01), dx * f)
    assert torch.equal(mc.conv3d_dgrad_skip(d, dy, w, add, ref, 0.01), (dx + add) * f)
    # a corner's infinity and NaN, and an infinite weight of a corner tap, which misses the volume at the other border
    x[0, 0, 0, 0, 0], x[-1, -1, -1, -1, 1] = float("inf"), float("nan")
    dy[0, 0, 0, 0, 1] = float("-inf")
    w[1, 0, 0, 2, 3] = float("inf")
    g = oc.shape(*case)
    xh, wh, dyh = (t.cpu().numpy() for t in (x, w, dy))
    for got, want in ((mc.conv3d_fwd(d, x, w), oc.fwd(g, xh, wh)), (mc.conv3d_dgrad(d, dy, w), oc.dgrad(g, dyh, wh)), (mc.conv3d_wgrad(d, x, dy), oc.wgrad(g, xh, dyh))):
        got = parity.to_host(got)
        for q in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(q(got), q(want)), (int(q(got).sum()), int(q(want).sum()))
