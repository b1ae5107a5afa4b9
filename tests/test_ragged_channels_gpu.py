"""bf16 layers whose channel counts no matrix-core kernel takes: operands padded to multiples of 32 (first layer: 4 input
channels), against the fp64 oracle on every element, and the plain kernels where the caller's workspace has no room."""
import ctypes

import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import conv3d as oc
from paper_1812_07816_amd import conv3d as mc
from paper_1812_07816_amd._lib import lib
from tests import parity

pytestmark = pytest.mark.gpu

PAD = "mfma_via_channel_padding"
CASES = [
    # N, D, H, W, Cin, Cout, k, s, p, kernels (None: whatever the dispatcher takes)
    (1, 5, 9, 13, 48, 48, 3, 1, 1, (PAD,) * 3),          # both counts padded, rows of whole 16-byte pieces
    (2, 4, 7, 11, 40, 24, 3, 1, 1, (PAD,) * 3),
    (1, 3, 17, 33, 33, 65, 3, 1, 0, (PAD,) * 3),         # odd counts: element by element, one channel into the next tile
    (1, 4, 6, 9, 32, 48, 3, 1, 2, (PAD,) * 3),           # only the output channels
    (2, 4, 6, 9, 31, 32, 3, 1, 1, (PAD,) * 3),           # only the input channels
    (1, 6, 19, 37, 3, 32, 3, 1, 1, (PAD,) * 3),          # padded to 4: first-layer kernels
    (2, 5, 9, 35, 1, 40, 3, 1, 1, (PAD,) * 3),
    (1, 4, 5, 34, 4, 8, 3, 1, 1, (PAD,) * 3),            # 4 input channels as they are
    (1, 7, 9, 13, 24, 72, 3, 2, 1, (PAD,) * 3),          # stride 2: output channels in 32s, as at stride 1
    (2, 8, 6, 10, 48, 96, 3, 2, 0, (PAD,) * 3),
    (1, 6, 8, 10, 32, 96, 3, 2, 1, ("mfma_stride2_plane_stream", "mfma_dgrad_stride2_parity", "mfma_wgrad_stride2")),
    (1, 4, 6, 8, 24, 48, 2, 2, 0, (PAD,) * 3),           # up-sampling layer
    (1, 1, 1, 1, 5, 7, 3, 1, 1, (PAD,) * 3),             # one voxel
    (1, 4, 4, 4, 40, 5, 1, 1, 0, ("direct",) * 3),       # 1x1x1: no kernel behind the padding
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[4]}-{c[5]}-k{c[6]}s{c[7]}" for c in CASES])
def test_ragged_channels_match_oracle(device, case):
    N, D, H, W, Cin, Cout, k, s, p, names = case
    desc = mc.make_desc(N, D, H, W, Cin, Cout, k, s, p, torch.bfloat16)
    assert tuple(mc.kernel_name(desc, q) for q in range(3)) == names
    errs = parity.run_case(95, 10 * CASES.index(case), N, D, H, W, Cin, Cout, k, s, p, bf16=True, full=True)
    for q, v in errs.items():
        assert v <= parity.TOL["bf16"], (case, q, v)


def test_plain_kernels_run_where_the_workspace_has_no_room_for_padding(device):
    """A caller that passes the workspace the plain kernels need (none for the forward pass and the data gradient) is
    served; so is the weight gradient that takes none, when the padded copies exceed its static scratch."""
    N, D, H, W, Cin, Cout = 1, 4, 6, 9, 40, 24
    x, w, dy = si.conv_case(95, 500, N, D, H, W, Cin, Cout, 3, 1, 1, True)
    g = oc.shape(N, D, H, W, Cin, Cout, 3, 1, 1)
    desc = mc.make_desc(N, D, H, W, Cin, Cout, 3, 1, 1, torch.bfloat16)
    xd, wd, dyd = (parity.to_device(a, True) for a in (x, w, dy))
    y, dx = torch.empty_like(dyd), torch.empty_like(xd)
    assert lib().mi3d_conv3d_fwd(ctypes.byref(desc), xd.data_ptr(), wd.data_ptr(), y.data_ptr(), None, 0, None) == 0
    assert lib().mi3d_conv3d_dgrad(ctypes.byref(desc), dyd.data_ptr(), wd.data_ptr(), dx.data_ptr(), None, 0, None) == 0
    torch.cuda.synchronize()
    assert oc.rel_err(parity.to_host(y), oc.fwd(g, x, w)) <= 1e-2
    assert oc.rel_err(parity.to_host(dx), oc.dgrad(g, dy, w)) <= 1e-2
    big = mc.make_desc(1, 64, 96, 96, 36, 40, 3, 1, 1, torch.bfloat16)      # (36 channels: behind the padding; in eights they need no copies)
    assert mc.workspace_bytes(big, mc.PASS_WGRAD) > mc.static_scratch_bytes()
    xb = torch.randn((1, 64, 96, 96, 36), device="cuda").bfloat16()
    dyb = torch.randn((1, 64, 96, 96, 40), device="cuda").bfloat16()
    got = torch.full((40, 3, 3, 3, 36), float("nan"), device="cuda")
    mc.conv3d_wgrad_static(big, xb, dyb, got)
    ref = mc.conv3d_wgrad(big, xb, dyb)      # on the matrix cores; both sum 590 000 products in fp32
    assert float((got - ref).norm() / ref.norm()) <= 1e-5
