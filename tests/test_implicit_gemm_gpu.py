"""The implicit GEMM for deep layers (small volumes at stride 1, many channels at stride 2) against the fp64 oracle, at
the sizes where its tiles can go wrong: positions that end inside a tile and tiles that span samples, channel counts
that end inside a step or a tile, extents of one, classes of the stride-2 data gradient without voxels, contractions
split and whole, and operands in two halves that meet inside a step."""
import ctypes

import pytest
import torch

from paper_1812_07816_amd import conv3d as mc
from paper_1812_07816_amd._lib import lib
from tests import parity

pytestmark = pytest.mark.gpu

CASES = [
    # N, D, H, W, Cin, Cout, s, p, contraction of the forward pass and of the data gradient (None: another kernel)
    (1, 1, 1, 1, 96, 96, 1, 1, "parts", "parts"),        # one voxel; 1.5 steps of channels per tap
    (3, 2, 2, 2, 320, 320, 1, 1, "parts", "parts"),      # a tile of positions spans three samples, contraction split many times
    (2, 5, 7, 9, 160, 32, 1, 1, "parts", None),          # half a tile of output channels
    (1, 6, 11, 13, 96, 224, 1, 0, "parts", "parts"),     # no padding: 128-wide tiles with 3/4 of the last in use
    (1, 4, 9, 9, 128, 192, 1, 2, "parts", "parts"),      # padding 2: outputs larger than the input
    (2, 9, 10, 11, 64, 96, 2, 1, "parts", "parts"),      # stride 2, odd and even extents, 1.5 steps contracted in the data gradient's tile
    (1, 1, 5, 1, 64, 128, 2, 1, "parts", "whole"),       # extents of one: six parity classes without a voxel
    (1, 11, 13, 12, 96, 128, 2, 0, "parts", "whole"),    # stride 2 without padding: the classes' taps are the other way round
    (1, 33, 31, 35, 64, 192, 2, 1, "parts", "whole"),
    (2, 31, 33, 64, 64, 128, 2, 1, "whole", "whole"),    # whole contractions (no partial sums) both ways
    (3, 4, 5, 40, 96, 96, 1, 0, "parts", "parts"),       # data gradient at positions beyond dy in rows, planes and samples of one tile
    (2, 6, 20, 21, 96, 128, 2, 0, "parts", "whole"),     # tiles that end one sample and begin the next, whose planes lie four on
    (2, 5, 24, 23, 128, 128, 1, 0, "parts", "parts"),
]


def _contraction(desc, q):
    name = mc.kernel_detail(desc, q)
    return None if not name.startswith("implicit_gemm") else "whole" if name.endswith("parts 1") else "parts"


@pytest.mark.parametrize("case", CASES)
def test_implicit_gemm_matches_oracle(device, case):
    N, D, H, W, Cin, Cout, s, p = case[:8]
    desc = mc.make_desc(N, D, H, W, Cin, Cout, 3, s, p, torch.bfloat16)
    assert (_contraction(desc, mc.PASS_FWD), _contraction(desc, mc.PASS_DGRAD)) == case[8:]
    # bf16 results: one rounding (2^-9 relative) of fp32 sums of at most 8640 products
    errs = parity.run_case(95, 600 + 10 * CASES.index(case), N, D, H, W, Cin, Cout, 3, s, p, bf16=True, full=True, passes=("fwd", "dgrad"))
    for q, v in errs.items():
        assert v <= parity.TOL["bf16"], (case, q, v)


@pytest.mark.parametrize("case", [(1, 4, 6, 8, 192, 96), (2, 3, 5, 7, 320, 192)])
def test_halves_that_meet_inside_a_step_give_the_same_bits(device, case):
    """Halves of 96 and 160 channels: a step of 64 channels begins in one tensor and ends in the other."""
    N, D, H, W, Cin, Cout = case
    desc = mc.make_desc(N, D, H, W, Cin, Cout, 3, 1, 1, torch.bfloat16)
    gen = torch.Generator(device="cuda").manual_seed(5)
    x, w, dy = (torch.randn(shape, generator=gen, device="cuda").bfloat16() for shape in
                ((N, D, H, W, Cin), (Cout, 3, 3, 3, Cin), (N, D, H, W, Cout)))
    assert _contraction(desc, mc.PASS_FWD) and _contraction(desc, mc.PASS_DGRAD)
    lo, hi = x[..., :Cin // 2].contiguous(), x[..., Cin // 2:].contiguous()
    assert torch.equal(mc.conv3d_fwd_pair(desc, lo, hi, w), mc.conv3d_fwd(desc, x, w))
    dlo, dhi = torch.empty_like(lo), torch.empty_like(hi)
    mc.conv3d_dgrad_pair(desc, dy, w, dlo, dhi)
    assert torch.equal(torch.cat([dlo, dhi], dim=-1), mc.conv3d_dgrad(desc, dy, w))


@pytest.mark.parametrize("case", [(1, 5, 800, 790, 64, 256, 1), (2, 4, 810, 800, 64, 256, 0)])
def test_planes_of_many_voxels(device, case):
    """Planes of 81 MB and more: the buffers move with the tap.  A tile ends one plane and begins the next, or (without
    padding) ends a sample whose last plane no position reads."""
    N, D, H, W, Cin, Cout, p = case
    desc = mc.make_desc(N, D, H, W, Cin, Cout, 3, 2, p, torch.bfloat16)
    assert [mc.kernel_detail(desc, q) for q in (0, 1)] == ["implicit_gemm_128x128_wide parts 1", "implicit_gemm_64x256_wide parts 1"]
    errs = parity.run_case(95, 900 + p, N, D, H, W, Cin, Cout, 3, 2, p, bf16=True, full=False, n_samples=20000, passes=("fwd", "dgrad"))
    for q, v in errs.items():
        assert v <= parity.TOL["bf16"], (case, q, v)


# geometry, pass, workspace that the query reported when these layers had kernels of their own
KEPT = [
    ((1, 8, 8, 8, 32, 96, 3, 1, 1), mc.PASS_DGRAD, 370688),
    ((1, 8, 8, 8, 96, 96, 3, 1, 1), mc.PASS_DGRAD, 1095680),
    ((1, 9, 10, 11, 256, 96, 3, 1, 1), mc.PASS_FWD, 4376576),
    ((1, 10, 10, 10, 64, 128, 3, 2, 1), mc.PASS_FWD, 578560),
]


@pytest.mark.parametrize("case", KEPT, ids=[f"{c[0][4]}-{c[0][5]}s{c[0][7]}" for c in KEPT])
def test_less_workspace_means_fewer_parts(device, case):
    """A workspace between the minimum and what the best split wants is enough, one byte less than the minimum is not; the
    result differs from the one with all parts by the order of the fp32 sums: one rounding to bf16."""
    args, q, kept = case
    desc = mc.make_desc(*args, torch.bfloat16)
    least, want = mc.min_workspace_bytes(desc, q), mc.workspace_bytes(desc, q)
    assert least <= kept < want
    parts = [int(mc.kernel_detail(desc, q, n).split("implicit_gemm_128x128 parts ")[1]) for n in (want, kept, least)]
    assert parts[0] > parts[1] > parts[2] == 1
    N, D, H, W, Cin, Cout = args[:6]
    gen = torch.Generator(device="cuda").manual_seed(9)
    out = (N, *mc.out_dims(desc), Cout)
    a = torch.randn(out if q == mc.PASS_DGRAD else (N, D, H, W, Cin), generator=gen, device="cuda").bfloat16()
    w = (torch.randn((Cout, 3, 3, 3, Cin), generator=gen, device="cuda") / 30).bfloat16()
    f = lib().mi3d_conv3d_dgrad if q == mc.PASS_DGRAD else lib().mi3d_conv3d_fwd
    got = []
    for n in (want, kept, least):
        o = torch.full((N, D, H, W, Cin) if q == mc.PASS_DGRAD else out, float("nan"), device="cuda").bfloat16()
        ws = torch.zeros(max(n, 16), dtype=torch.uint8, device="cuda")
        assert f(ctypes.byref(desc), a.data_ptr(), w.data_ptr(), o.data_ptr(), ws.data_ptr() if n else None, n, None) == 0, n
        torch.cuda.synchronize()
        got.append(o.float())
    for o in got[1:]:
        assert float((o - got[0]).abs().max()) <= 2.0 ** -8 * float(got[0].abs().max())
    if least:
        assert f(ctypes.byref(desc), a.data_ptr(), w.data_ptr(), o.data_ptr(), ws.data_ptr(), least - 1, None) == -3
