"""Weight gradient as a matrix product over numbered positions, bf16 and fp32 (products from bf16 matrix instructions): tails of
tiles and steps, every form of stride, splits of the positions, halves and values the parts cannot hold."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import conv3d as oc
from paper_1812_07816_amd import conv3d as mc
from tests import parity

pytestmark = pytest.mark.gpu

# fp32 sums of n terms of random sign: an accumulator is rounded three times per 32 positions (bf16: four), at most 2048 steps
# follow each other: sqrt(3 * 2048) half roundings of 2^-24 are 2.3e-6 of the result's root mean square for one standard deviation
# of the worst order; ten of those
TOL = 3e-5

CASES = [
    # N, D, H, W, Cin, Cout, k, s, p, bf16
    (1, 12, 12, 12, 64, 320, 3, 1, 1, True),      # last tile of rows half full
    (2, 4, 4, 4, 256, 96, 3, 1, 1, True),
    (1, 3, 7, 5, 96, 32, 3, 1, 2, True),          # padding 2, few rows
    (2, 2, 2, 2, 320, 64, 3, 1, 1, True),         # less than a step of positions
    (3, 9, 11, 13, 64, 160, 3, 2, 1, True),       # odd extents, stride 2
    (2, 8, 10, 12, 32, 64, 3, 2, 0, True),
    (1, 18, 20, 20, 2, 8, 3, 1, 1, False),        # one tile of columns
    (2, 6, 9, 11, 20, 44, 3, 2, 0, False),
    (2, 5, 9, 13, 32, 130, 3, 2, 1, False),       # two rows in the last tile
    (1, 9, 8, 7, 64, 80, 3, 1, 2, False),
    (1, 5, 7, 9, 30, 126, 2, 2, 0, False),         # voxels no position reads
    (2, 8, 8, 8, 160, 96, 3, 1, 1, False),
    (1, 1, 1, 1, 64, 64, 3, 1, 1, False),
]


def _uses(d, ws=None):
    return "wgrad_implicit_gemm" in mc.kernel_detail(d, mc.PASS_WGRAD, ws)


def _desc(case):
    *geo, bf16 = case
    return mc.make_desc(*geo, torch.bfloat16 if bf16 else torch.float32)


@pytest.mark.parametrize("case", CASES, ids=[f"{c[1]}x{c[2]}x{c[3]}-{c[4]}-{c[5]}k{c[6]}s{c[7]}p{c[8]}{'b' if c[9] else 'f'}" for c in CASES])
def test_matches_oracle_with_every_workspace(device, case):
    """With the workspace of the query, with room for fewer splits of the positions, and with the least."""
    *geo, bf16 = case
    d = _desc(case)
    assert _uses(d)
    x, w, dy = si.conv_case(94, 10 * CASES.index(case), *geo, bf16)
    ref = oc.wgrad(oc.shape(*geo), x, dy)
    xd, dyd = parity.to_device(x, bf16), parity.to_device(dy, bf16)
    want, least = mc.workspace_bytes(d, 2), mc.min_workspace_bytes(d, 2)
    for n in sorted({want, (want + least) // 2, least}):
        ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")[:n]
        dw = torch.full((geo[5],) + (geo[6],) * 3 + (geo[4],), 7.0, device="cuda")
        mc.conv3d_wgrad(d, xd, dyd, dw, ws)
        assert oc.rel_err(parity.to_host(dw), ref) <= TOL, (n, mc.kernel_detail(d, 2, n))
    again = mc.conv3d_wgrad(d, xd, dyd)
    assert torch.equal(again, mc.conv3d_wgrad(d, xd, dyd))


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("Cin", [64, 128, 320])
def test_halves(device, Cin, bf16):
    """The two halves of a virtual concatenation, at different distances from each other."""
    case = (2, 4, 5, 6, Cin, 64, 3, 1, 1, bf16)
    d, dt = _desc(case), torch.bfloat16 if bf16 else torch.float32
    assert _uses(d) and mc.pair_supported(d, 2)
    torch.manual_seed(1)
    x, dy = torch.randn((2, 4, 5, 6, Cin), device="cuda").to(dt), torch.randn((2, 4, 5, 6, 64), device="cuda").to(dt)
    hi = x[..., Cin // 2:].contiguous()
    lo = x[..., :Cin // 2].contiguous()
    ref = mc.conv3d_wgrad(d, x, dy)
    for a, b in ((lo, hi), (lo, hi.clone())):
        got = mc.conv3d_wgrad_pair(d, a, b, dy)
        assert float((got - ref).double().norm() / ref.double().norm()) <= 1e-6


@pytest.mark.parametrize("k, s, p", [((1, 2, 2), (1, 2, 2), 0), ((3, 3, 3), (1, 2, 2), 1), ((2, 3, 1), (2, 1, 1), (0, 1, 0))])
def test_axes_of_their_own(device, k, s, p):
    g = torch.Generator().manual_seed(3)
    x = torch.randn((2, 72, 6, 9, 10), generator=g).double()
    d = mc.make_desc(2, 6, 9, 10, 72, 136, k, s, p, torch.float32)
    assert _uses(d)
    dy = torch.randn((2, 136, *mc.out_dims(d)), generator=g).double()
    ref = torch.nn.grad.conv3d_weight(x, (136, 72, *k), dy, stride=s, padding=p).permute(0, 2, 3, 4, 1)
    dev = lambda t: t.permute(0, 2, 3, 4, 1).float().contiguous().cuda()
    got = mc.conv3d_wgrad(d, dev(x), dev(dy)).cpu().double()
    assert float((got - ref).abs().max() / ref.square().mean().sqrt()) <= TOL


@pytest.mark.parametrize("where", ["x", "dy", "large", "tiny", "scaled"])
@pytest.mark.parametrize("case", [(2, 5, 6, 9, 64, 96, 3, 1, 1), (2, 9, 8, 11, 20, 64, 3, 2, 1), (1, 6, 8, 10, 32, 160, 2, 2, 0), (1, 4, 5, 6, 12, 140, 3, 1, 2)])
def test_values_without_parts(device, case, where):
    """Infinities and NaN reach exactly the elements whose sums hold them; what the parts cannot hold keeps its precision."""
    N, D, H, W, Cin, Cout, k, s, p = case
    x, w, dy = si.conv_case(94, 700 + Cin, *case, False)
    if where in ("x", "dy"):
        a = x if where == "x" else dy
        a[0, 0, 0, 0, 0], a[0, -1, -1, -1, 1], a[N - 1, 1, -1, 0, -1] = np.inf, -np.inf, np.nan
    elif where == "large":         # rounds to infinity in bf16
        x[0, 1, 2, 3, 4] = 3.4e38
        dy *= np.float32(1e-3)
    elif where == "tiny":          # parts below the normal range
        x *= np.float32(2.0 ** -112)
    else:                          # products of ordinary size from large and small values
        x *= np.float32(2.0 ** 115); dy *= np.float32(2.0 ** -75)
    d, g = _desc((*case, False)), oc.shape(*case)
    assert _uses(d)
    got, ref = parity.to_host(mc.conv3d_wgrad(d, parity.to_device(x, False), parity.to_device(dy, False))), oc.wgrad(g, x, dy)
    for f in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(f(got), f(ref)), (int(f(got).sum()), int(f(ref).sum()))
    ok = np.isfinite(ref)
    gv, rv = got[ok].astype(np.float64), ref[ok].astype(np.float64)
    rms = np.sqrt(np.mean(rv * rv)) if where != "large" else np.median(np.abs(rv))
    assert np.max(np.abs(gv - rv) / np.maximum(np.abs(rv), rms)) <= TOL
