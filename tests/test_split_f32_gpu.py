"""fp32 3x3x3 convolutions whose products come from bf16 matrix instructions (each operand in three parts): edges of the
tiles and of the dispatch rule against the fp64 oracle, and values the parts cannot hold against the fp32 instructions,
which a call with the smaller workspace gets."""
import ctypes
import itertools

import pytest
import torch

import synth_inputs as si
from oracle import conv3d as oc
from paper_1812_07816_amd import conv3d as mc
from paper_1812_07816_amd._lib import lib
from tests import parity

pytestmark = pytest.mark.gpu

# fp32 sums of n terms of random sign: about sqrt(n) half roundings of 2^-24, n = 27 * 320 at most: 6e-6 of the result's
# root mean square for one standard deviation of the worst operand order; five of those
TOL = 3e-5

CASES = [
    # N, D, H, W, Cin, Cout, k, s, p; passes whose products come from bf16 parts
    ((1, 3, 9, 33, 16, 16, 3, 1, 1), "01"),       # one stage deep, one row and column beyond an 8 x 32 tile
    ((1, 2, 17, 48, 48, 33, 3, 1, 1), "0"),      # 16 x 16 tiles, one channel beyond a block of 32
    ((2, 3, 7, 31, 32, 80, 3, 1, 0), "01"),       # row-major tiles, no padding, last block of 64 half full
    ((1, 3, 5, 12, 64, 5, 3, 1, 2), "0"),        # padding 2, few output channels
    ((1, 4, 1, 1, 32, 16, 3, 1, 1), "01"),        # one column: planes above and below are zero
    ((1, 2, 200, 1, 32, 16, 3, 1, 1), "01"),    # patch of a one-column plane too large: the implicit GEMM
    ((1, 3, 12, 12, 320, 320, 3, 1, 1), "01"),    # deepest level
    ((1, 5, 11, 13, 32, 64, 3, 2, 1), "01"),     # parity classes of an odd extent (forward: the implicit GEMM)
    ((2, 4, 6, 70, 16, 64, 3, 2, 0), "01"),      # no padding: classes with one and two taps change places
    ((2, 49, 41, 65, 32, 32, 3, 1, 1), "012"),     # weight gradient: one row and column beyond its 4 x 32 patches
    ((1, 55, 30, 31, 64, 96, 3, 1, 0), "012"),
    ((3, 30, 15, 28, 96, 64, 3, 1, 2), "012"),     # padding 2: dy planes beyond both ends
    ((1, 6, 8, 34, 16, 32, (1, 3, 3), 1, (0, 1, 1)), "01"),   # one plane per output
]


@pytest.mark.parametrize("case, parts", CASES, ids=[f"{c[1]}x{c[2]}x{c[3]}-{c[4]}-{c[5]}s{c[7]}" for c, _ in CASES])
def test_split_products_match_oracle(device, case, parts):
    N, D, H, W, Cin, Cout, k, s, p = case
    d = mc.make_desc(N, D, H, W, Cin, Cout, k, s, p, torch.float32)
    assert "".join(str(q) for q in range(3) if mc.kernel_detail(d, q).endswith("from_bf16_parts")) == parts
    if isinstance(k, tuple):
        x = torch.randn((N, D, H, W, Cin), device="cuda")
        w = torch.randn((Cout, *k, Cin), device="cuda")
        ref = torch.nn.functional.conv3d(x.cpu().double().permute(0, 4, 1, 2, 3), w.cpu().double().permute(0, 4, 1, 2, 3), padding=p)
        err = mc.conv3d_fwd(d, x, w).cpu().double() - ref.permute(0, 2, 3, 4, 1)
        assert float(err.abs().max() / ref.square().mean().sqrt()) <= TOL
        return
    errs = parity.run_case(97, 10 * CASES.index((case, parts)), N, D, H, W, Cin, Cout, k, s, p, bf16=False, full=True)
    for q in ("fwd", "dgrad", "wgrad"):
        assert errs[q] <= TOL, (case, q, errs)


def _both(d, q, a, w, shape):
    """The pass with the workspace the query reports and with what the fp32 instructions need."""
    K, M = (d.Cout, d.Cin) if q == mc.PASS_DGRAD else (d.Cin, d.Cout)
    small = (27 * K * ((M + 31) // 32 * 32) * 4 + 255) // 256 * 256
    assert mc.workspace_bytes(d, q) > small
    assert (mc.kernel_detail(d, q), mc.kernel_detail(d, q, small)) == ("f32_gather_from_bf16_parts", "f32_gather")
    f = lib().mi3d_conv3d_dgrad if q == mc.PASS_DGRAD else lib().mi3d_conv3d_fwd
    outs = []
    for n in (mc.workspace_bytes(d, q), small):
        ws, o = torch.zeros(n, dtype=torch.uint8, device="cuda"), torch.empty(shape, device="cuda")
        assert f(ctypes.byref(d), a.data_ptr(), w.data_ptr(), o.data_ptr(), ws.data_ptr(), n, None) == 0
        torch.cuda.synchronize()
        outs.append(o)
    return outs


@pytest.mark.parametrize("q", [0, 1], ids=["fwd", "dgrad"])
@pytest.mark.parametrize("kind", ["inf", "nan", "large", "tiny", "tiny_w", "inf_w", "scaled", "overflow", "ends", "subnormal"])
def test_values_without_parts_take_the_fp32_instructions(device, kind, q):
    torch.manual_seed(5)
    d = mc.make_desc(1, 3, 10, 40, 32, 48, 3, 1, 1, torch.float32)
    K, M = (48, 32) if q == mc.PASS_DGRAD else (32, 48)
    a, w = torch.randn((1, 3, 10, 40, K), device="cuda"), torch.randn((48, 3, 3, 3, 32), device="cuda")
    if kind == "inf":
        a[0, 1, 3, 5, 17], a[0, 2, 9, 39, 3] = float("inf"), float("-inf")
    elif kind == "nan":
        a[0, 0, 0, 33, 31] = float("nan")
    elif kind == "large":          # rounds to infinity in bf16; the products stay finite
        a[0, 1, 2, 3, 4] = 3.4e38
        w *= 1e-3
    elif kind == "tiny":           # parts below the normal range
        a *= 2.0 ** -112
    elif kind == "tiny_w":
        w *= 2.0 ** -112
    elif kind == "inf_w":
        w[3, 1, 2, 0, 7] = float("inf")
    elif kind == "scaled":         # products of ordinary size from large and small values
        a *= 2.0 ** 115
        w *= 2.0 ** -75
    elif kind == "overflow":       # every product overflows, to an infinity of the output channel's sign
        a = a.abs().clamp(min=0.1) * 1e21
        w = w.abs().clamp(min=0.1) * 1e21
        w[(..., slice(None, None, 2)) if q == mc.PASS_DGRAD else slice(None, None, 2)] *= -1
    elif kind == "ends":           # the ends of what the parts hold
        a *= 2.0 ** 42
        w *= 2.0 ** -80
    else:                          # products of the small parts are subnormal numbers
        a *= 2.0 ** -62
        w *= 2.0 ** -64
    got, ref = _both(d, q, a, w, (1, 3, 10, 40, M))
    for f in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(f(got), f(ref)), kind
    ok = torch.isfinite(ref)
    if kind == "overflow":
        assert torch.isinf(ref).all()
        return
    g, r = got[ok].double(), ref[ok].double()
    rms = r.square().mean().sqrt() if kind != "large" else r.abs().median()
    assert float(((g - r).abs() / torch.maximum(r.abs(), rms)).max()) <= TOL


@pytest.mark.parametrize("tap", [(0, 0, 0), (1, 1, 1), (2, 1, 0), (1, 2, 2)])
def test_weight_without_parts_in_a_class_of_the_strided_data_gradient(device, tap):
    """Each parity class runs its own taps: the one with the weight must take the fp32 instructions, in its stage."""
    torch.manual_seed(7)
    d = mc.make_desc(1, 5, 10, 13, 32, 64, 3, 2, 1, torch.float32)
    dy, w = torch.randn((1, 3, 5, 7, 64), device="cuda"), torch.randn((64, 3, 3, 3, 32), device="cuda")
    w[(37, *tap, 9)] = float("inf")
    got, ref = _both(d, mc.PASS_DGRAD, dy, w, (1, 5, 10, 13, 32))
    for f in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(f(got), f(ref))
    ok = torch.isfinite(ref)
    assert not ok.all() and float((got[ok] - ref[ok]).abs().max() / ref[ok].square().mean().sqrt()) <= TOL


def _weight_gradient(x, dy):
    """dw of a 3x3x3 layer with padding 1 in 64 bits, over the window alone: what is not finite is added voxel by voxel."""
    x, dy = x.double().cpu(), dy.double().cpu()
    xf, dyf = (torch.where(torch.isfinite(v), v, 0.0).permute(0, 4, 1, 2, 3) for v in (x, dy))
    ref = torch.nn.grad.conv3d_weight(xf, (dy.shape[-1], x.shape[-1], 3, 3, 3), dyf, padding=1).permute(0, 2, 3, 4, 1).clone()
    ext = x.shape[1:4]
    for t in itertools.product(range(3), repeat=3):
        for n, *i, c in (~torch.isfinite(x)).nonzero().tolist():
            o = [v + 1 - k for v, k in zip(i, t)]
            if all(0 <= v < e for v, e in zip(o, ext)):
                ref[:, t[0], t[1], t[2], c] += x[n, i[0], i[1], i[2], c] * dy[n, o[0], o[1], o[2], :]
        for n, *o, c in (~torch.isfinite(dy)).nonzero().tolist():
            i = [v - 1 + k for v, k in zip(o, t)]
            if all(0 <= v < e for v, e in zip(i, ext)):
                ref[c, t[0], t[1], t[2], :] += dy[n, o[0], o[1], o[2], c] * x[n, i[0], i[1], i[2], :]
    return ref


@pytest.mark.parametrize("kind", ["inf", "nan_dy", "border", "border_dy", "large", "tiny", "scaled", "overflow", "ends", "subnormal"])
def test_weight_gradient_of_values_without_parts(device, kind):
    """Columns that end inside a patch of 32, rows inside one of 4."""
    torch.manual_seed(6)
    N, D, H, W, c = 2, 96, 22, 60, 32
    d = mc.make_desc(N, D, H, W, c, c, 3, 1, 1, torch.float32)
    assert mc.kernel_detail(d, mc.PASS_WGRAD) == "f32_wgrad_from_bf16_parts"
    x, dy = torch.randn((N, D, H, W, c), device="cuda"), torch.randn((N, D, H, W, c), device="cuda")
    if kind == "inf":
        x[0, 3, 5, 7, 11], x[1, 10, 13, 31, 31] = float("inf"), float("-inf")
    elif kind == "nan_dy":
        dy[1, 1, 1, 33, 2] = float("nan")
    elif kind == "border":
        x[0, 0, 0, 0, 11], x[1, 95, 21, 59, 31] = float("inf"), float("-inf")
    elif kind == "border_dy":
        dy[0, 95, 0, 59, 3], dy[1, 0, 21, 31, 30] = float("inf"), float("nan")
    elif kind == "large":
        x[0, 6, 9, 9, 4] = 3.4e38
        dy *= 1e-3
    elif kind == "tiny":
        x *= 2.0 ** -112
    elif kind == "scaled":
        x *= 2.0 ** 115
        dy *= 2.0 ** -75
    elif kind == "overflow":
        x = x.abs().clamp(min=0.1) * 1e21
        dy = dy.abs().clamp(min=0.1) * 1e21
        dy[..., ::2] *= -1
    elif kind == "ends":
        x *= 2.0 ** 42
        dy *= 2.0 ** -80
    else:
        x *= 2.0 ** -62
        dy *= 2.0 ** -64
    got = mc.conv3d_wgrad(d, x, dy).double().cpu()
    if kind == "overflow":
        sign = torch.tensor([-1.0, 1.0], dtype=torch.float64).repeat(c // 2)
        assert torch.equal(got, (sign * float("inf"))[:, None, None, None, None].expand_as(got))
        return
    ref = _weight_gradient(x, dy)
    for f in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(f(got), f(ref)), kind
    ok = torch.isfinite(ref)
    g, r = got[ok], ref[ok]
    rms = r.square().mean().sqrt() if kind != "large" else r.abs().median()
    assert float(((g - r).abs() / torch.maximum(r.abs(), rms)).max()) <= TOL


def test_worst_operands_of_the_split(device):
    """1 + 2^-8 - 2^-17 has parts 1, 2^-8 and -2^-17: the products left out are 2^-24 of the product, all of one sign.  Sums of
    the rest are multiples of 2^-7.  With 32 channels, and in the weight gradient of 64, whose small products are added
    apart, every addition is exact and what is left out is the whole error; with 64 the forward sums pass 1024, where six
    roundings of at most 2^-24 per 16 of the 27 x 64 products come on top."""
    v, N, D, H, W = 1 + 2.0 ** -8 - 2.0 ** -17, 2, 24, 22, 60
    one = torch.ones((N, 1, D, H, W), dtype=torch.float64)
    window = torch.nn.functional.conv3d(one, torch.ones((1, 1, 3, 3, 3), dtype=torch.float64), padding=1).permute(0, 2, 3, 4, 1)
    overlap = torch.nn.grad.conv3d_weight(one, (1, 1, 3, 3, 3), one, padding=1).permute(0, 2, 3, 4, 1)
    for c, most in ((32, 1), (64, 1 + 6 * 27 * 4)):
        d = mc.make_desc(N, D, H, W, c, c, 3, 1, 1, torch.float32)
        assert (mc.kernel_detail(d, mc.PASS_WGRAD) == "f32_wgrad_from_bf16_parts") == (c == 64)
        x, w = torch.full((N, D, H, W, c), v, device="cuda"), torch.full((c, 3, 3, 3, c), v, device="cuda")
        for got, r, m in ((mc.conv3d_fwd(d, x, w), c * v * v * window, most), (mc.conv3d_dgrad(d, x, w), c * v * v * window, most),
                          (mc.conv3d_wgrad(d, x, x), v * v * overlap, 1)):
            assert float(((got.double().cpu() - r) / r).abs().max()) <= m * 2.0 ** -24, c
