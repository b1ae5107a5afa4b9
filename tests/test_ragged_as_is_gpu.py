"""bf16 3x3x3 layers with channel counts in multiples of 8 that 32 does not divide, on the kernels over numbered positions without
padding: strides, paddings, steps of (tap, channel) pairs and of 64 channels, tiles of 32 and more channels, every workspace from
the query's down, and values that are not finite, against the fp64 oracle on every element."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import conv3d as oc
from paper_1812_07816_amd import conv3d as mc
from tests import parity

pytestmark = pytest.mark.gpu

CASES = [
    # N, D, H, W, Cin, Cout, k, s, p (1024 output voxels at least: smaller volumes are padded but for the weight gradient)
    (1, 9, 11, 13, 48, 48, 3, 1, 1),
    (2, 7, 9, 11, 24, 104, 3, 1, 2),      # a last block of 8 channels; positions beyond the volume they read from
    (1, 12, 13, 14, 8, 24, 3, 1, 0),      # eight taps per step, less than a block of 32 channels
    (1, 11, 12, 13, 64, 40, 3, 1, 1),     # forward pass in steps of 64 channels
    (1, 11, 12, 13, 40, 64, 3, 1, 1),     # data gradient in steps of 64 channels
    (1, 11, 12, 13, 32, 48, 3, 1, 1),
    (1, 35, 30, 1, 40, 48, 3, 1, 1),      # one column
    (2, 17, 18, 19, 48, 40, 3, 2, 1),     # eight classes of one to eight taps in steps of pairs
    (2, 18, 17, 20, 24, 64, 3, 2, 0),     # in steps of 64 channels, no padding
    (2, 17, 18, 19, 96, 40, 3, 2, 1),     # half a step of 64 channels
    (1, 23, 21, 25, 104, 8, 3, 2, 1),
    (1, 2, 64, 70, 8, 8, 3, 2, 1),
]
IDS = [f"{c[1]}x{c[2]}x{c[3]}-{c[4]}-{c[5]}s{c[7]}p{c[8]}" for c in CASES]


def _workspaces(d, q):
    """The query's, with room for the flags of the weights but whole contractions, and the least of this path."""
    want = mc.workspace_bytes(d, q)
    if q == mc.PASS_WGRAD:
        return sorted({want, want // 2, 0}, reverse=True)
    copy = (d.Cin * d.Cout * 27 * 2 + 255) // 256 * 256 if q == mc.PASS_DGRAD else 0     # of the weights
    return sorted({want, min(want, copy + 1024), copy}, reverse=True)


def _run(d, q, x, w, dy, n):
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")[:n]
    if q == mc.PASS_FWD:
        return mc.conv3d_fwd(d, x, w, torch.full_like(dy, float("nan")), ws)
    if q == mc.PASS_DGRAD:
        return mc.conv3d_dgrad(d, dy, w, torch.full_like(x, float("nan")), ws)
    return mc.conv3d_wgrad(d, x, dy, torch.full(w.shape, float("nan"), device="cuda"), ws)


@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_matches_oracle_with_every_workspace(device, case):
    d, g = mc.make_desc(*case, torch.bfloat16), oc.shape(*case)
    x, w, dy = si.conv_case(99, 10 * CASES.index(case), *case, True)
    refs = oc.fwd(g, x, w), oc.dgrad(g, dy, w), oc.wgrad(g, x, dy)
    dev = [parity.to_device(a, True) for a in (x, w, dy)]
    for q in range(3):
        for n in _workspaces(d, q):
            how = mc.kernel_detail(d, q, n)
            assert how.startswith("wgrad_implicit_gemm" if q == 2 else "implicit_gemm"), how
            err = oc.rel_err(parity.to_host(_run(d, q, *dev, n)), refs[q])
            print(case, q, n, how, f"{err:.2e}", flush=True)
            # (a weight gradient is not rounded to bf16: sums of fp32, as test_wgrad_positions_gpu.py bounds them)
            assert err <= (3e-5 if q == 2 else parity.TOL["bf16"]), (case, q, n, how, err)


@pytest.mark.parametrize("where", ["x", "dy", "w"])
@pytest.mark.parametrize("case", [CASES[i] for i in (1, 3, 7, 8, 9)], ids=[IDS[i] for i in (1, 3, 7, 8, 9)])
def test_values_that_are_not_finite_reach_their_windows_alone(device, case, where):
    N = case[0]
    d, g = mc.make_desc(*case, torch.bfloat16), oc.shape(*case)
    x, w, dy = si.conv_case(99, 500 + 10 * CASES.index(case), *case, True)
    a = {"x": x, "dy": dy, "w": w}[where]
    if where == "w":
        a[1, 0, 0, 2, case[4] // 2], a[case[5] - 1, 2, 0, 0, 0] = np.inf, np.nan
    else:
        a[0, 0, 0, 0, 0], a[0, -1, -1, -1, 1], a[N - 1, 1, -1, 0, a.shape[-1] - 1] = np.inf, -np.inf, np.nan
    dev = [parity.to_device(v, True) for v in (x, w, dy)]
    for q, other, ref in ((0, "dy", oc.fwd(g, x, w)), (1, "x", oc.dgrad(g, dy, w)), (2, "w", oc.wgrad(g, x, dy))):
        if where == other:
            continue
        for n in _workspaces(d, q):
            got = parity.to_host(_run(d, q, *dev, n))
            for f in (np.isnan, np.isposinf, np.isneginf):
                assert np.array_equal(f(got), f(ref)), (case, q, n, int(f(got).sum()), int(f(ref).sum()))
            ok = np.isfinite(ref)
            assert ok.any() and oc.rel_err(got[ok], ref[ok]) <= parity.TOL["bf16"], (case, q, n)


def _at(x, w, vox):
    """Outputs of the stride-1 layer with padding 1 at voxels [n, 3] of the only sample, in fp64; w as [Cout, 3, 3, 3, Cin]."""
    ext = torch.tensor(x.shape[1:4], device="cuda")
    acc = torch.zeros((len(vox), w.shape[0]), dtype=torch.float64, device="cuda")
    for t in np.ndindex(3, 3, 3):
        at = vox + torch.tensor(t, device="cuda") - 1
        ok = ((at >= 0) & (at < ext)).all(1)
        c = at.clamp(min=0).minimum(ext - 1)
        acc += (x[0, c[:, 0], c[:, 1], c[:, 2]].double() * ok[:, None]) @ w[(slice(None), *t)].double().T
    return acc


@pytest.mark.parametrize("C", [8, 24])
def test_layers_whose_padded_copies_would_pass_16_gib(device, C):
    """24 channels: tensors of more than 4 GiB as well (the weight gradient addresses up to that)."""
    D, H, W = 512, 512, 520
    d = mc.make_desc(1, D, H, W, C, C, 3, 1, 1, torch.bfloat16)
    gen = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn((1, D, H, W, C), generator=gen, device="cuda", dtype=torch.bfloat16)
    w = torch.randn((C, 3, 3, 3, C), generator=gen, device="cuda", dtype=torch.bfloat16)
    assert all(mc.kernel_detail(d, q).startswith("implicit_gemm") and mc.workspace_bytes(d, q) < 1 << 20 for q in (0, 1))
    ends = torch.cartesian_prod(*(torch.tensor([0, 1, e // 2, e - 2, e - 1]) for e in (D, H, W))).cuda()
    vox = torch.cat([ends, (torch.rand((3000, 3), generator=gen, device="cuda") * torch.tensor([D, H, W], device="cuda")).long()])
    flipped = w.flip((1, 2, 3)).permute(4, 1, 2, 3, 0)
    for got, ref in ((mc.conv3d_fwd(d, x, w), _at(x, w, vox)), (mc.conv3d_dgrad(d, x, w), _at(x, flipped, vox))):
        e = got[0, vox[:, 0], vox[:, 1], vox[:, 2]].double() - ref
        assert float((e.abs() / torch.maximum(ref.abs(), ref.square().mean().sqrt())).max()) <= parity.TOL["bf16"]
        del got
    if C == 8:
        assert mc.kernel_detail(d, 2).startswith("wgrad_implicit_gemm")
        dy = torch.zeros_like(x)             # a few voxels at both ends and between, so that the sum is formed again
        dy[0, vox[:200, 0], vox[:200, 1], vox[:200, 2]] = torch.randn((200, C), generator=gen, device="cuda", dtype=torch.bfloat16)
        dw, ref = mc.conv3d_wgrad(d, x, dy).double(), torch.zeros((C, 3, 3, 3, C), dtype=torch.float64, device="cuda")
        u = torch.unique(vox[:200], dim=0)
        for t in np.ndindex(3, 3, 3):
            at = u + torch.tensor(t, device="cuda") - 1
            ok = ((at >= 0) & (at < torch.tensor([D, H, W], device="cuda"))).all(1)
            at = at[ok]
            ref[(slice(None), *t)] = dy[0, u[ok][:, 0], u[ok][:, 1], u[ok][:, 2]].double().T @ x[0, at[:, 0], at[:, 1], at[:, 2]].double()
        assert float((dw - ref).abs().max() / ref.square().mean().sqrt()) <= 3e-5


@pytest.mark.parametrize("args, q", [((1, 66, 66, 67, 16, 96, 3, 1, 1), 1), ((1, 66, 66, 67, 96, 16, 3, 1, 1), 0), ((2, 52, 53, 51, 24, 96, 3, 1, 1), 0),
                                     ((1, 90, 91, 92, 32, 48, 3, 2, 1), 0), ((1, 89, 80, 79, 64, 24, 3, 2, 1), 1), ((1, 60, 61, 62, 128, 24, 3, 1, 1), 2)])
def test_padded_and_as_they_are(device, args, q):
    """Layers beyond the lines of the dispatch: behind the padding with the workspace of the query, as they are with too little for the copies."""
    d = mc.make_desc(*args, torch.bfloat16)
    gen = torch.Generator(device="cuda").manual_seed(5)
    xs, ws, ys = mc._shapes(d)
    x, w, dy = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in (xs, ws, ys))
    small = (27 * d.Cin * d.Cout * 2 + 255) // 256 * 256 if q < 2 else 16 << 20
    assert mc.kernel_detail(d, q).startswith("padded_channels") and "padded" not in mc.kernel_detail(d, q, small)
    a, b = (_run(d, q, x, w, dy, n).double() for n in (mc.workspace_bytes(d, q), small))
    # each rounds to bf16 once (weight gradients: fp32 sums of 113460 products at most, in other orders)
    assert float((a - b).norm() / a.norm()) <= (3e-6 if q == 2 else 2.0 ** -8)
