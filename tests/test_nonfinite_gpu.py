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
