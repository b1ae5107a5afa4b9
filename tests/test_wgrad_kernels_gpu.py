"""Weight-gradient kernels on patches, at sizes that the product over numbered positions leaves to them: the stride-2 kernel with
32 and 64 output channels a workgroup, columns taken two patch rows at a time, and the fp32 instructions; odd extents, padding 0
to 2, patches that end outside the volume.  Against the fp64 oracle (large volumes: a sample of the elements)."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import conv3d as oc
from paper_1812_07816_amd import conv3d as mc
from tests import parity

pytestmark = pytest.mark.gpu

S2, PLANES, F32 = "mfma_wgrad_stride2", "mfma_wgrad_plane_stream", "f32_wgrad"
CASES = [
    # N, D, H, W, Cin, Cout, k, s, p
    (S2, (1, 51, 55, 130, 32, 32, 3, 2, 0)),
    (S2, (2, 70, 21, 115, 32, 32, 3, 2, 1)),
    (S2, (1, 141, 33, 190, 32, 32, 3, 2, 0)),     # one column beyond the third patch
    (S2, (1, 177, 93, 63, 32, 64, 3, 2, 0)),
    (S2, (1, 107, 67, 121, 32, 64, 3, 2, 1)),
    (S2, (1, 46, 73, 62, 64, 32, 3, 2, 0)),
    (S2, (2, 63, 24, 63, 64, 32, 3, 2, 1)),
    (S2, (1, 86, 105, 64, 64, 128, 3, 2, 0)),
    (S2, (2, 101, 15, 64, 128, 128, 3, 2, 1)),
    (PLANES, (1, 26, 24, 48, 32, 32, 3, 1, 1)),   # a last column of 16, two patch rows
    (PLANES, (1, 21, 38, 50, 32, 32, 3, 1, 0)),   # three: the last pair is half empty
    (PLANES, (3, 3, 36, 46, 32, 32, 3, 1, 2)),
    (PLANES, (2, 19, 48, 16, 32, 32, 3, 1, 1)),   # no other column
    (PLANES, (3, 14, 48, 14, 32, 32, 3, 1, 2)),
    (PLANES, (1, 9, 60, 46, 64, 64, 3, 1, 1)),
    (PLANES, (1, 3, 22, 44, 64, 128, 3, 1, 2)),
    (PLANES, (2, 19, 18, 16, 256, 128, 3, 1, 1)),
    (PLANES, (1, 40, 47, 61, 64, 64, 3, 1, 1)),   # 16-row patches
    (F32, (1, 3, 5, 6, 33, 35, 3, 1, 0)),
    (F32, (1, 8, 4, 3, 33, 35, 3, 1, 1)),
    (F32, (1, 7, 3, 3, 33, 35, 3, 2, 1)),
    (F32, (1, 30, 29, 31, 33, 35, 3, 1, 1)),
    (F32, (1, 16, 20, 19, 7, 9, 3, 1, 0)),
    (F32, (1, 8, 27, 19, 5, 48, 3, 1, 1)),
    (F32, (1, 9, 4, 6, 64, 33, 2, 2, 0)),
    (F32, (1, 3, 23, 42, 31, 64, 2, 1, 1)),
    (F32, (2, 5, 21, 37, 32, 31, 3, 2, 1)),
]


@pytest.mark.parametrize("how, case", CASES, ids=[f"{c[1]}x{c[2]}x{c[3]}-{c[4]}-{c[5]}k{c[6]}s{c[7]}p{c[8]}" for _, c in CASES])
def test_matches_oracle(device, how, case):
    d = mc.make_desc(*case, torch.float32 if how == F32 else torch.bfloat16)
    assert mc.kernel_detail(d, mc.PASS_WGRAD) == how
    small = d.N * d.D * d.H * d.W * d.Cin * d.Cout < 3e7
    errs = parity.run_case(94, 5000 + 10 * CASES.index((how, case)), *case, bf16=how != F32, passes=("wgrad",), full=small, n_wgrad_samples=400)
    # fp32 sums of up to a million products of random sign in at most 256 parts: a thousand half roundings of 2^-24 at random
    assert errs["wgrad"] <= 3e-5, errs


@pytest.mark.parametrize("case", [(3, 14, 48, 14, 32, 32, 3, 1, 2), (1, 3, 22, 44, 64, 128, 3, 1, 2), (2, 63, 24, 63, 64, 32, 3, 2, 1),
                                  (4, 14, 22, 9, 256, 32, 3, (1, 2, 2), 1), (1, 46, 73, 62, 50, 32, 3, 2, 0)],
                         ids=["planes", "planes_wide", "strided", "unit_stride", "padded"])
def test_without_room_for_the_partial_sums(device, case):
    """A call with less than the kernel on patches asks for runs the product over positions, down to the least workspace."""
    d = mc.make_desc(*case, torch.bfloat16)
    want, least = mc.workspace_bytes(d, 2), mc.min_workspace_bytes(d, 2)
    assert mc.kernel_detail(d, 2).split(" > ")[-1] in (S2, PLANES)
    x, w, dy = si.conv_case(94, 5900 + want % 1000, *case, True)
    g = oc.shape(*case)
    xd, dyd = parity.to_device(x, True), parity.to_device(dy, True)
    at = np.random.default_rng(7).integers(0, 27 * d.Cin * d.Cout, 300)
    ref = oc.wgrad_at(g, x, dy, at)
    for n in (want - 256, (want + least) // 2 // 256 * 256, least):
        assert "wgrad_implicit_gemm" in mc.kernel_detail(d, 2, n) or (case[4] == 50 and n < want - 256), n   # (no room for the padded copies)
        ws = torch.empty(n + 16, dtype=torch.uint8, device="cuda")[:n]
        dw = torch.full((d.Cout, 3, 3, 3, d.Cin), 7.0, device="cuda")
        mc.conv3d_wgrad(d, xd, dyd, dw, ws)
        # (one part: a chain of at most 20000 steps of 32 positions, rounded half a step of 2^-24 at random each)
        assert parity._sampled_err(parity.to_host(dw).ravel()[at], ref) <= 3e-5, n
