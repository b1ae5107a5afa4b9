"""Infinities and NaN reach exactly the results whose window holds them: against the fp64 oracle, which adds up the products
inside the window and nothing else.  A kernel that adds zeros of its own (padding, unused columns) turns 0 x inf into NaN."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import conv3d as oc
from paper_1812_07816_amd import conv3d as mc
from tests import parity

pytestmark = pytest.mark.gpu


def _same(got, ref, tol, what):
    """Same NaN and infinities; finite values within the tolerance of the repository's parity tests."""
    for f in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(f(got), f(ref)), (what, int(f(got).sum()), int(f(ref).sum()))
    ok = np.isfinite(ref)
    assert ok.any(), what
    assert oc.rel_err(got[ok], ref[ok]) <= tol, what


FIRST = [
    # N, D, H, W, Cin, Cout, p
    (1, 5, 9, 40, 4, 32, 1),
    (2, 4, 18, 67, 4, 64, 0),
    (1, 5, 9, 40, 3, 32, 1),
    (1, 4, 17, 35, 1, 32, 2),
    (1, 5, 9, 40, 4, 24, 1),
    (1, 4, 9, 33, 2, 40, 1),
]


@pytest.mark.parametrize("case", FIRST, ids=[f"{c[4]}-{c[5]}p{c[6]}" for c in FIRST])
def test_first_layer_forward_keeps_to_its_window(device, case):
    """Four columns are contracted for a window of three: the fourth must not be read."""
    N, D, H, W, Cin, Cout, p = case
    x, w, _ = si.conv_case(98, 10 * FIRST.index(case), N, D, H, W, Cin, Cout, 3, 1, p, True)
    x[0, 2, 3, 5, 0], x[0, 1, 8, 20, Cin - 1], x[N - 1, D - 1, 5, W - 1, 0] = np.inf, -np.inf, np.nan
    desc = mc.make_desc(N, D, H, W, Cin, Cout, 3, 1, p, torch.bfloat16)
    y = parity.to_host(mc.conv3d_fwd(desc, parity.to_device(x, True), parity.to_device(w, True)))
    _same(y, oc.fwd(oc.shape(N, D, H, W, Cin, Cout, 3, 1, p), x, w), parity.TOL["bf16"], case)


RAGGED = [
    # N, D, H, W, Cin, Cout, k, s, p
    (1, 5, 9, 13, 48, 48, 3, 1, 1),      # both counts padded
    (2, 4, 7, 35, 40, 24, 3, 1, 1),
    (1, 4, 9, 33, 33, 65, 3, 1, 0),      # element by element
    (1, 3, 6, 9, 32, 48, 3, 1, 2),       # data gradient without slicing
    (2, 4, 6, 9, 31, 32, 3, 1, 1),       # forward pass without slicing
    (1, 4, 9, 34, 3, 40, 3, 1, 1),       # four input channels
    (1, 4, 9, 34, 3, 32, 3, 1, 1),       # forward pass without slicing, four input channels
    (1, 4, 5, 34, 4, 24, 3, 1, 1),       # data gradient without slicing, four input channels
    (1, 7, 9, 13, 24, 72, 3, 2, 1),
    (2, 8, 6, 10, 48, 96, 3, 2, 0),
    (1, 5, 6, 7, 40, 40, 3, (1, 2, 2), 1),   # unit-stride embedding behind the padding
    (1, 4, 6, 8, 24, 48, 2, 2, 0),
    (1, 4, 6, 8, 24, 24, 2, 2, 0),
    (1, 4, 4, 4, 264, 64, 2, 2, 0),      # 3x3x3 embedding behind the padding, forward pass without slicing
]


@pytest.mark.parametrize("where", ["x", "dy", "w"])
@pytest.mark.parametrize("case", RAGGED, ids=[f"{c[4]}-{c[5]}k{c[6]}s{c[7]}p{c[8]}" for c in RAGGED])
def test_padded_channels_sum_over_the_window_alone(device, case, where):
    """Values at the ends of the volume, where the window of some results and the zero filling of the kernels meet."""
    N, D, H, W, Cin, Cout, k, s, p = case
    x, w, dy = si.conv_case(98, 500 + 10 * RAGGED.index(case), N, D, H, W, Cin, Cout, k, s, p, True)
    a = {"x": x, "dy": dy, "w": w}[where]
    if where == "w":
        a[1, 0, 0, k - 1, Cin // 2], a[Cout - 1, k - 1, 0, 0, 0] = np.inf, np.nan
    else:
        a[0, 0, 0, 0, 0], a[0, -1, -1, -1, 1], a[N - 1, 1, -1, 0, a.shape[-1] - 1] = np.inf, -np.inf, np.nan
    desc = mc.make_desc(N, D, H, W, Cin, Cout, k, s, p, torch.bfloat16)
    g = oc.shape(N, D, H, W, Cin, Cout, k, s, p)
    xd, wd, dyd = (parity.to_device(v, True) for v in (x, w, dy))
    tol = parity.TOL["bf16"]
    if where != "dy":
        _same(parity.to_host(mc.conv3d_fwd(desc, xd, wd)), oc.fwd(g, x, w), tol, ("fwd", case))
    if where != "x":
        _same(parity.to_host(mc.conv3d_dgrad(desc, dyd, wd)), oc.dgrad(g, dy, w), tol, ("dgrad", case))
    if where != "w":
        _same(parity.to_host(mc.conv3d_wgrad(desc, xd, dyd)), oc.wgrad(g, x, dy), tol, ("wgrad", case))


@pytest.mark.parametrize("case", [(2, 4, 6, 9, 31, 32, 3, 1, 1), (1, 3, 6, 9, 32, 48, 3, 1, 2)])
def test_padding_without_room_for_the_flags(device, case):
    """The least workspace of a padded layer holds no flags of the weights: every result is looked at instead."""
    N, D, H, W, Cin, Cout, k, s, p = case
    q = mc.PASS_FWD if Cin % 32 else mc.PASS_DGRAD
    x, w, dy = si.conv_case(98, 900 + Cin, N, D, H, W, Cin, Cout, k, s, p, True)
    w[1, 0, 0, k - 1, Cin // 2] = np.inf
    desc = mc.make_desc(N, D, H, W, Cin, Cout, k, s, p, torch.bfloat16)
    g = oc.shape(N, D, H, W, Cin, Cout, k, s, p)
    ws = torch.empty(mc.workspace_bytes(desc, q) - 256, dtype=torch.uint8, device="cuda")
    xd, wd, dyd = (parity.to_device(v, True) for v in (x, w, dy))
    got, ref = ((mc.conv3d_fwd(desc, xd, wd, ws=ws), oc.fwd(g, x, w)) if q == mc.PASS_FWD else
                (mc.conv3d_dgrad(desc, dyd, wd, ws=ws), oc.dgrad(g, dy, w)))
    _same(parity.to_host(got), ref, parity.TOL["bf16"], case)
