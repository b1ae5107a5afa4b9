"""fp32 layers as an implicit GEMM over numbered positions (products from bf16 matrix instructions): tails of the tiles and of
the steps, every form of stride, splits of the contraction, epilogues and values the parts cannot hold."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import conv3d as oc
from paper_1812_07816_amd import conv3d as mc
from tests import parity

pytestmark = pytest.mark.gpu

# fp32 sums of n terms of random sign: about sqrt(n) half roundings of 2^-24, n = 27 * 320 at most: 6e-6 of the result's
# root mean square for one standard deviation of the worst operand order; five of those
TOL = 3e-5

CASES = [
    # N, D, H, W, Cin, Cout, k, s, p; passes that take the kernel
    ((1, 4, 6, 8, 32, 64, 2, 2, 0), "01"),        # taps as output channels, one tile
    ((2, 5, 7, 9, 60, 108, 2, 2, 0), "01"),        # odd extents: voxels no tap reaches, channels that end inside a block
    ((1, 3, 16, 17, 64, 44, 2, 2, 0), "01"),
    ((2, 6, 9, 11, 20, 44, 3, 2, 0), "01"),       # classes with one to eight taps, steps that span taps
    ((2, 13, 14, 15, 32, 64, 3, 2, 1), "01"),
    ((1, 9, 8, 7, 40, 48, 3, 1, 2), "0"),         # padding 2
    ((1, 6, 7, 5, 64, 36, 3, 1, 1), "01"),        # more splits than tiles
    ((2, 3, 4, 5, 20, 700, 1, 1, 0), "01"),         # less than a step
    ((1, 7, 6, 9, 8, 200, 2, 1, 1), "01"),         # even extent, unit stride
    ((1, 1, 1, 1, 64, 132, 3, 1, 1), "01"),       # one voxel
    ((1, 2, 200, 1, 32, 16, 3, 1, 1), "01"),      # one column
    ((3, 5, 5, 5, 4, 128, 3, 1, 1), "01"),          # eight taps per step
    ((1, 11, 12, 9, 128, 320, 3, 1, 1), "01"),
    ((1, 4, 4, 4, 640, 96, 3, 2, 1), "01"),       # many steps, few positions
]


def _uses(d, q, ws=None):
    return mc.kernel_detail(d, q, ws).startswith("f32_implicit_gemm")


@pytest.mark.parametrize("case, passes", CASES, ids=[f"{c[1]}x{c[2]}x{c[3]}-{c[4]}-{c[5]}k{c[6]}s{c[7]}p{c[8]}" for c, _ in CASES])
def test_matches_oracle(device, case, passes):
    N, D, H, W, Cin, Cout, k, s, p = case
    d = mc.make_desc(N, D, H, W, Cin, Cout, k, s, p, torch.float32)
    assert "".join(str(q) for q in range(2) if _uses(d, q)) == passes
    errs = parity.run_case(95, 10 * CASES.index((case, passes)), N, D, H, W, Cin, Cout, k, s, p, bf16=False, passes=("fwd", "dgrad"), full=True)
    assert max(errs.values()) <= TOL, (case, errs)


@pytest.mark.parametrize("k, s, p", [((1, 2, 2), (1, 2, 2), 0), ((3, 3, 3), (1, 2, 2), 1), ((2, 3, 1), (2, 1, 1), (0, 1, 0)), ((3, 1, 2), (1, 1, 2), (1, 0, 0))])
def test_axes_of_their_own(device, k, s, p):
    g = torch.Generator().manual_seed(3)
    x = torch.randn((2, 72, 6, 9, 10), generator=g, dtype=torch.float64)
    w = torch.randn((136, 72, *k), generator=g, dtype=torch.float64)
    d = mc.make_desc(2, 6, 9, 10, 72, 136, k, s, p, torch.float32)
    assert _uses(d, 0) and _uses(d, 1)
    y = torch.nn.functional.conv3d(x.float().double(), w.float().double(), stride=s, padding=p)
    dy = torch.randn(y.shape, generator=g, dtype=torch.float64)
    dx = torch.nn.grad.conv3d_input(x.shape, w.float().double(), dy.float().double(), stride=s, padding=p)
    dev = lambda t: t.permute(0, 2, 3, 4, 1).float().contiguous().cuda()
    for got, ref in ((mc.conv3d_fwd(d, dev(x), dev(w)), y), (mc.conv3d_dgrad(d, dev(dy), dev(w)), dx)):
        e = got.cpu().double().permute(0, 4, 1, 2, 3) - ref
        assert float(e.abs().max() / ref.square().mean().sqrt()) <= TOL


@pytest.mark.parametrize("case", [(2, 6, 7, 9, 64, 40, 3, 1, 1), (2, 8, 7, 10, 64, 96, 3, 2, 1), (1, 8, 10, 6, 32, 64, 2, 2, 0)])
def test_smaller_workspaces(device, case):
    """Fewer splits of the contraction, none, and the fp32 instructions."""
    N, D, H, W, Cin, Cout, k, s, p = case
    d = mc.make_desc(N, D, H, W, Cin, Cout, k, s, p, torch.float32)
    xs, wsh, ys = mc._shapes(d)
    torch.manual_seed(1)
    x, w, dy = torch.randn(xs, device="cuda"), torch.randn(wsh, device="cuda"), torch.randn(ys, device="cuda")
    for q in (0, 1):
        want, least = mc.workspace_bytes(d, q), mc.min_workspace_bytes(d, q)
        seen, outs = set(), []
        for n in sorted({want, (want + least) // 2, least + (want - least) // 8, least}, reverse=True):
            seen.add(mc.kernel_detail(d, q, n))
            ws = torch.empty(n, dtype=torch.uint8, device="cuda")
            outs.append((mc.conv3d_fwd(d, x, w, ws=ws) if q == 0 else mc.conv3d_dgrad(d, dy, w, ws=ws)).double())
        assert _uses(d, q) and not _uses(d, q, least) and len(seen) > 1
        for o in outs[1:]:
            assert float((o - outs[0]).abs().max() / outs[0].square().mean().sqrt()) <= TOL


@pytest.mark.parametrize("case", [(2, 5, 6, 7, 64, 64, 3, 1, 1), (1, 40, 38, 36, 64, 128, 3, 2, 1), (2, 6, 7, 9, 64, 96, 3, 2, 1), (1, 9, 8, 11, 64, 32, 2, 2, 0)])
def test_epilogues_and_halves(device, case):
    """Fused epilogues and the two halves of a virtual concatenation against the same pass without them."""
    N, D, H, W, Cin, Cout, k, s, p = case
    d = mc.make_desc(N, D, H, W, Cin, Cout, k, s, p, torch.float32)
    xs, wsh, ys = mc._shapes(d)
    torch.manual_seed(2)
    x, w, dy, add, ref = (torch.randn(v, device="cuda") for v in (xs, wsh, ys, xs, xs))
    assert _uses(d, 0) and _uses(d, 1)
    y, dx = mc.conv3d_fwd(d, x, w), mc.conv3d_dgrad(d, dy, w)
    lo, hi = (x[..., i * Cin // 2:(i + 1) * Cin // 2].contiguous() for i in (0, 1))
    assert torch.equal(mc.conv3d_fwd_pair(d, lo, hi, w), y)
    assert torch.equal(torch.cat(mc.conv3d_dgrad_pair(d, dy, w), -1), dx)
    leaky = lambda t: torch.where(t > 0, t, 0.01 * t)
    assert torch.equal(mc.conv3d_fwd_lrelu(d, x, w, 0.01), leaky(y))
    f = torch.where(ref > 0, 1.0, 0.01)
    assert torch.equal(mc.conv3d_dgrad_lrelu(d, dy, w, ref, 0.01), dx * f)
    assert torch.equal(mc.conv3d_dgrad_skip(d, dy, w, add, ref, 0.01), (dx + add) * f)


@pytest.mark.parametrize("where", ["x", "w", "dy", "large", "tiny", "scaled"])
@pytest.mark.parametrize("case", [(2, 5, 6, 9, 64, 40, 3, 1, 1), (2, 9, 8, 11, 20, 64, 3, 2, 1), (1, 5, 8, 7, 32, 64, 2, 2, 0), (1, 3, 4, 6, 12, 140, 3, 1, 2)])
def test_values_without_parts(device, case, where):
    """Infinities and NaN reach exactly the results whose window holds them; what the parts cannot hold keeps its precision."""
    N, D, H, W, Cin, Cout, k, s, p = case
    x, w, dy = si.conv_case(95, 700 + Cin, N, D, H, W, Cin, Cout, k, s, p, False)
    if where in ("x", "dy"):
        a = x if where == "x" else dy
        a[0, 0, 0, 0, 0], a[0, -1, -1, -1, 1], a[N - 1, 1, -1, 0, -1] = np.inf, -np.inf, np.nan
    elif where == "w":
        w[1, 0, 0, k - 1, Cin // 2], w[Cout - 1, k - 1, 0, 0, 0] = np.inf, np.nan
    elif where == "large":         # rounds to infinity in bf16
        x[0, 1, 2, 3, 4], dy[0, 1, 1, 1, 4] = 3.4e38, -3.4e38
        w *= np.float32(1e-3)
    elif where == "tiny":          # parts below the normal range
        x *= np.float32(2.0 ** -112); dy *= np.float32(2.0 ** -112)
    else:                          # products of ordinary size from large and small values
        x *= np.float32(2.0 ** 115); dy *= np.float32(2.0 ** 115); w *= np.float32(2.0 ** -75)
    d, g = mc.make_desc(N, D, H, W, Cin, Cout, k, s, p, torch.float32), oc.shape(N, D, H, W, Cin, Cout, k, s, p)
    xd, wd, dyd = (parity.to_device(v, False) for v in (x, w, dy))
    for q, got, ref in ((0, mc.conv3d_fwd(d, xd, wd), oc.fwd(g, x, w)), (1, mc.conv3d_dgrad(d, dyd, wd), oc.dgrad(g, dy, w))):
        if not _uses(d, q):
            continue
        got = parity.to_host(got)
        for f in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(f(got), f(ref)), (q, int(f(got).sum()), int(f(ref).sum()))
        ok = np.isfinite(ref)
        gv, rv = got[ok].astype(np.float64), ref[ok].astype(np.float64)
        rms = np.sqrt(np.mean(rv * rv)) if where != "large" else np.median(np.abs(rv))
        assert np.max(np.abs(gv - rv) / np.maximum(np.abs(rv), rms)) <= TOL
