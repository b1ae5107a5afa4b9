"""Data gradients of the implicit GEMM that read the weights as they are, transposing them on the way out of LDS, against
the fp64 oracle: every width of a row of weights in LDS, channels that end inside a tile, contractions that end inside a
step (their rows lie behind the end of the weights), and no workspace where the contraction is whole."""
import pytest
import torch

from paper_1812_07816_amd import conv3d as mc
from tests import parity

pytestmark = pytest.mark.gpu

CASES = [
    # N, D, H, W, Cin, Cout, s, rows of a tile
    (1, 17, 16, 18, 32, 96, 2, 32),       # rows of 64 bytes; 1.5 steps
    (1, 19, 15, 18, 32, 320, 2, 32),
    (1, 61, 62, 60, 64, 160, 2, 64),      # rows of 128 bytes; 2.5 steps
    (1, 6, 7, 8, 224, 128, 1, 128),       # rows of 256 bytes; 3/4 of the last tile's in use
    (2, 6, 5, 6, 96, 192, 1, 128),
    (2, 3, 4, 5, 320, 96, 2, 128),
]


@pytest.mark.parametrize("case", CASES)
def test_matches_oracle(device, case):
    N, D, H, W, Cin, Cout, s, rows = case
    desc = mc.make_desc(N, D, H, W, Cin, Cout, 3, s, 1, torch.bfloat16)
    assert mc.kernel_detail(desc, mc.PASS_DGRAD).startswith("implicit_gemm_%dx" % rows), mc.kernel_detail(desc, mc.PASS_DGRAD)
    assert mc.min_workspace_bytes(desc, mc.PASS_DGRAD) == 0
    # one rounding to bf16 (2^-9 relative) of fp32 sums of at most 8640 products
    errs = parity.run_case(97, 700 + CASES.index(case), N, D, H, W, Cin, Cout, 3, s, 1, bf16=True, full=True, passes=("dgrad",))
    assert all(v <= parity.TOL["bf16"] for v in errs.values()), (case, errs)


def test_values_that_must_not_spread(device):
    """An infinite weight of the last output channel and zeros behind it: only the voxels it reaches are not finite."""
    desc = mc.make_desc(1, 6, 6, 6, 96, 128, 3, 1, 1, torch.bfloat16)
    w = torch.ones((128, 3, 3, 3, 96), device="cuda").bfloat16()
    w[127, 1, 1, 1, 95] = float("inf")
    dy = torch.zeros((1, 6, 6, 6, 128), device="cuda").bfloat16()
    dy[0, 2, 3, 4, 127] = 1.0
    dy += 0.25
    dx = mc.conv3d_dgrad(desc, dy, w)
    bad = ~torch.isfinite(dx.float())
    assert int(bad.sum()) == 216 and bool(bad[..., 95].all())   # (every voxel's own dy meets the centre tap of that channel)
