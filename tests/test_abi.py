"""The C-ABI library loads and exports every symbol include/mi3d.h declares
(no compute calls; runs without a GPU)."""
import ctypes
import os
import re

from paper_1812_07816_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    src = open(os.path.join(ROOT, "include", "mi3d.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(mi3d_[a-z0-9_]+)\s*\(", src)))


def test_header_declares_the_hot_path_calls():
    names = _declared()
    for n in ("mi3d_conv3d_fwd", "mi3d_conv3d_dgrad", "mi3d_conv3d_wgrad", "mi3d_swap_out", "mi3d_swap_in", "mi3d_swap_plan"):
        assert n in names


def test_library_exports_every_declared_symbol():
    l = ctypes.CDLL(_lib.LIB_PATH)
    for n in _declared():
        assert hasattr(l, n), n


def test_binding_covers_every_declared_symbol():
    assert sorted(_lib.SIGNATURES) == _declared()


def test_status_strings():
    l = _lib.lib()
    seen = set()
    for s in range(0, -8, -1):
        msg = l.mi3d_status_string(s)
        assert msg and msg not in seen
        seen.add(msg)
    assert l.mi3d_status_string(-99) == b"unknown status"


def test_descriptor_validation_needs_no_gpu():
    from paper_1812_07816_amd import conv3d as mc
    d = mc.make_desc(1, 192, 192, 192, 32, 64, 3, 2, 1, 1)
    assert mc.out_dims(d) == (96, 96, 96)
    a = ctypes.c_int()
    bad = mc.make_desc(1, 1, 4, 4, 1, 1, 3, 1, 0, 0)
    assert _lib.lib().mi3d_conv3d_out_dims(ctypes.byref(bad), ctypes.byref(a), ctypes.byref(a), ctypes.byref(a)) == -1
    bad = mc.make_desc(1, 4, 4, 4, 1, 1, 3, 1, 1, 7)
    assert _lib.lib().mi3d_conv3d_out_dims(ctypes.byref(bad), ctypes.byref(a), ctypes.byref(a), ctypes.byref(a)) == -2
    # null pointers are rejected before anything is launched
    assert _lib.lib().mi3d_conv3d_fwd(ctypes.byref(d), None, None, None, None, 0, None) == -1
    assert _lib.lib().mi3d_conv3d_fwd(None, None, None, None, None, 0, None) == -1


def test_largest_sizes_are_routed_by_their_plane_size_or_refused():
    """The tiled kernels address inside a D-plane with 32-bit offsets: a descriptor whose planes reach 2 GiB must go to
    the kernels with 64-bit indices, whatever its channel counts; one beyond 2^40 elements is refused outright.
    (Host logic only: nothing is launched.)"""
    import torch
    from paper_1812_07816_amd import conv3d as mc
    bf = torch.bfloat16
    # 64 GiB tensors with 64 MiB planes: still the tiled kernels
    d = mc.make_desc(1, 1024, 1024, 1024, 32, 32, 3, 1, 1, bf)
    assert [mc.kernel_name(d, q) for q in range(3)] == ["mfma_plane_stream", "mfma_plane_stream", "mfma_wgrad_plane_stream"]
    # the last plane size below the limit, and the first one at it
    d = mc.make_desc(1, 4, 4096, 4096, 32, 32, 3, 1, 1, bf)          # 1 GiB planes
    assert mc.kernel_name(d, 0) == "mfma_plane_stream"
    for args in ((1, 4, 8192, 8192, 32, 32, 3, 1, 1),     # stride 1, 4 GiB planes
                 (1, 4, 4096, 4096, 64, 64, 3, 1, 1),     # exactly 2 GiB
                 (1, 4, 8192, 4096, 32, 32, 3, 2, 1),     # stride 2: the input plane decides
                 (1, 4, 16384, 16384, 4, 32, 3, 1, 1)):   # first layer: the output plane decides
        d = mc.make_desc(*args, bf)
        assert [mc.kernel_name(d, q) for q in range(3)] == ["direct"] * 3, args
    a = ctypes.c_int()
    huge = mc.make_desc(64, 4096, 4096, 4096, 32, 32, 3, 1, 1, bf)   # 2^47 elements
    assert _lib.lib().mi3d_conv3d_out_dims(ctypes.byref(huge), ctypes.byref(a), ctypes.byref(a), ctypes.byref(a)) == -2


def test_strided_layers_keep_their_kernels_on_large_planes():
    """Up to the 2 GiB a plane that the tiled kernels address (64 channels: 4000 x 4000 voxels)."""
    import torch
    from paper_1812_07816_amd import conv3d as mc
    for hw in (700, 800, 1200, 2000, 4000):
        d = mc.make_desc(1, 8, hw, hw, 64, 128, 3, 2, 1, torch.bfloat16)
        assert [mc.kernel_name(d, q) for q in range(2)] == ["mfma_stride2_plane_stream", "mfma_dgrad_stride2_parity"], hw
    d = mc.make_desc(2, 9, 1200, 1200, 128, 256, 3, 2, 0, torch.bfloat16)
    assert [mc.kernel_name(d, q) for q in range(2)] == ["mfma_stride2_plane_stream", "mfma_dgrad_stride2_parity"]


def test_kernel_detail_names_what_runs_and_refuses_what_a_call_refuses():
    import torch
    from paper_1812_07816_amd import conv3d as mc
    d = mc.make_desc(1, 12, 12, 12, 320, 320, 3, 1, 1, torch.bfloat16)
    assert mc.kernel_detail(d, 0).startswith("implicit_gemm") and mc.kernel_detail(d, 0, 0).endswith("parts 1")
    d = mc.make_desc(1, 8, 8, 8, 40, 48, 3, 1, 1, torch.bfloat16)
    assert mc.kernel_detail(d, 0) == "padded_channels > plane_stream" and mc.kernel_detail(d, 0, 0) == "direct"
    d = mc.make_desc(1, 64, 64, 64, 64, 64, 3, 1, 1, torch.float32)
    least = mc.min_workspace_bytes(d, 1)
    assert mc.kernel_detail(d, 1) == "f32_gather_from_bf16_parts" and mc.kernel_detail(d, 1, least) == "f32_gather"
    for args in ((1, 48, 48, 48, 64, 128, 2, 2, 0), (2, 12, 14, 16, 32, 64, 3, 2, 1), (1, 10, 9, 8, 20, 44, 3, 1, 1)):   # (whatever the patch kernel takes)
        e = mc.make_desc(*args, torch.float32)
        assert mc.kernel_detail(e, 0).startswith("f32_implicit_gemm") and mc.kernel_detail(e, 0).endswith("_from_bf16_parts")
    buf = ctypes.create_string_buffer(64)
    l = _lib.lib()
    assert l.mi3d_conv3d_kernel_detail(ctypes.byref(d), 1, least - 1, buf, 64) == -3
    assert l.mi3d_conv3d_kernel_detail(ctypes.byref(d), 3, least, buf, 64) == -1
    assert l.mi3d_conv3d_kernel_detail(ctypes.byref(d), 1, least, None, 0) == -1
    assert l.mi3d_conv3d_kernel_detail(None, 1, least, buf, 64) == -1


def test_ragged_layers_ask_for_what_they_use():
    """3x3x3 with channels in eights: the layer is read as it is, so no pass wants room for copies of its tensors, and with the
    least its own kernels take (a copy of the weights for the data gradient, nothing else) it stays on them."""
    import torch
    from paper_1812_07816_amd import conv3d as mc
    for args in ((1, 128, 128, 128, 48, 48, 3, 1, 1), (1, 37, 50, 61, 48, 48, 3, 1, 1), (1, 47, 44, 47, 40, 72, 3, 1, 1), (2, 30, 31, 32, 24, 40, 3, 2, 1)):
        d = mc.make_desc(*args, torch.bfloat16)
        copy = (27 * d.Cin * d.Cout * 2 + 255) // 256 * 256
        assert all(mc.workspace_bytes(d, q) <= 64 << 20 for q in range(3)), args
        for q, least in ((0, 0), (1, copy), (2, 0)):
            for n in (least, mc.workspace_bytes(d, q)):
                assert mc.kernel_detail(d, q, n).startswith("wgrad_implicit_gemm" if q == 2 else "implicit_gemm"), (args, q, n, mc.kernel_detail(d, q, n))
    d = mc.make_desc(1, 64, 96, 96, 41, 40, 3, 1, 1, torch.bfloat16)      # not in eights: behind the padding
    assert mc.kernel_detail(d, 0) == "padded_channels > plane_stream"


def test_ragged_layers_are_padded_where_that_was_measured_to_be_faster():
    """One layer on either side of each line, and both ways for a caller whose workspace holds no copies."""
    import torch
    from paper_1812_07816_amd import conv3d as mc
    for args, q, padded in (((1, 103, 92, 115, 8, 96, 3, 1, 1), 1, True), ((1, 43, 53, 44, 8, 96, 3, 1, 1), 1, False),        # contracted channels whole
                            ((1, 72, 69, 58, 96, 16, 3, 1, 1), 0, True), ((1, 45, 50, 45, 96, 16, 3, 1, 1), 0, False),
                            ((1, 88, 89, 88, 24, 96, 3, 1, 1), 0, True), ((1, 98, 97, 96, 16, 64, 3, 1, 1), 0, False),        # outputs whole
                            ((1, 150, 100, 160, 48, 48, 3, 1, 1), 0, False), ((1, 150, 100, 160, 48, 48, 3, 1, 1), 1, False), # neither
                            ((1, 140, 131, 129, 32, 48, 3, 2, 1), 0, True), ((1, 140, 131, 129, 64, 48, 3, 2, 1), 0, False),  # stride 2
                            ((1, 89, 87, 111, 64, 24, 3, 2, 1), 1, True), ((1, 80, 60, 53, 64, 48, 3, 2, 1), 1, False),
                            ((1, 102, 101, 101, 64, 16, 3, 1, 1), 2, True), ((1, 37, 50, 61, 48, 48, 3, 1, 1), 2, False),
                            ((2, 40, 40, 40, 24, 48, 3, (1, 2, 2), 1), 2, False)):
        d = mc.make_desc(*args, torch.bfloat16)
        assert mc.kernel_detail(d, q).startswith("padded_channels") == padded, (args, q, mc.kernel_detail(d, q))
        assert "implicit_gemm" in mc.kernel_detail(d, q, 27 * 128 * 128 * 2), (args, q)


def test_the_smallest_fp32_weight_gradients_keep_to_their_line():
    """One launch of workgroups that fetch whole lines for a few channels, up to where the matrix product over positions is faster."""
    import torch
    from paper_1812_07816_amd import conv3d as mc
    for args, tiny in (((1, 18, 18, 18, 32, 64, 2, 2, 0), True), ((1, 24, 24, 24, 32, 64, 2, 2, 0), False), ((1, 40, 38, 32, 32, 64, 2, 2, 0), False),
                       ((1, 24, 24, 24, 32, 32, 2, 2, 0), True), ((1, 32, 32, 32, 32, 32, 2, 2, 0), False), ((1, 20, 20, 20, 32, 32, 1, 1, 0), False),
                       ((1, 20, 20, 20, 16, 16, 3, 1, 1), True), ((1, 20, 20, 20, 4, 8, 3, 1, 1), True), ((1, 32, 32, 32, 32, 16, 3, 2, 1), False)):
        how = mc.kernel_detail(mc.make_desc(*args, torch.float32), 2)
        assert how == "f32_direct" if tiny else "wgrad_implicit_gemm" in how, (args, how)


def test_narrow_planes_of_paired_patch_rows_keep_their_weight_gradient():
    """Planes of at most 16 columns are taken two patch rows at a time: the model of the patches' time counts them so."""
    import torch
    from paper_1812_07816_amd import conv3d as mc
    for args, how in (((2, 19, 18, 16, 256, 128, 3, 1, 1), "mfma_wgrad_plane_stream"), ((2, 19, 18, 17, 256, 128, 3, 1, 1), "wgrad_implicit_gemm"),
                      ((1, 12, 12, 12, 320, 320, 3, 1, 1), "wgrad_implicit_gemm")):
        assert mc.kernel_detail(mc.make_desc(*args, torch.bfloat16), 2).startswith(how), args


def test_plans_do_not_depend_on_what_was_asked_before():
    """A thread keeps its last plans: what runs, for which workspace, is the same in any order and in any thread."""
    import random
    import threading
    import torch
    from paper_1812_07816_amd import conv3d as mc
    r = random.Random(3)
    asks = []
    for _ in range(150):
        c = [r.choice([8, 24, 32, 64, 96, 256]) for _ in range(2)]
        k, s, p = r.choice([(3, 1, 1), (3, 2, 1), (2, 2, 0), (3, 1, 0)])
        dt = r.choice([torch.bfloat16, torch.float32])
        d = mc.make_desc(r.randint(1, 2), *(r.randint(4, 60) for _ in range(3)), *c, k, s, p, dt)
        for q in range(3):
            full = mc.workspace_bytes(d, q)
            asks += [(d, q, n) for n in {full, (full + mc.min_workspace_bytes(d, q)) // 2, mc.min_workspace_bytes(d, q)}]
    said = [mc.kernel_detail(*a) for a in asks]
    order = list(range(len(asks)))
    r.shuffle(order)
    wrong = []

    def again(idx):
        wrong.extend(i for i in idx if mc.kernel_detail(*asks[i]) != said[i])

    threads = [threading.Thread(target=again, args=(o,)) for o in (order, order[::-1], sorted(order))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    for d, q, n in (asks[i] for i in order[:60]):       # one size away, and back
        e = type(d).from_buffer_copy(d)
        e.W += 1
        first = mc.kernel_detail(d, q, n)
        mc.workspace_bytes(e, q)
        assert mc.kernel_detail(d, q, n) == first


def test_weight_gradients_run_in_the_workspace_that_earlier_builds_reported():
    """A saved size stays enough: layers that went back to the kernels on patches run in what the product over positions asked for."""
    import torch
    from paper_1812_07816_amd import conv3d as mc
    for args, before in (((1, 11, 18, 12, 256, 192, 3, 1, 2), 15925248), ((4, 12, 19, 15, 512, 160, 3, 1, 1), 17694720),
                         ((2, 44, 37, 49, 512, 64, 3, 2, 1), 14155776), ((4, 32, 35, 36, 128, 32, 3, 2, 1), 7962624),
                         ((4, 14, 22, 9, 256, 32, 3, (1, 2, 2), 1), 8672256),
                         ((1, 123, 73, 136, 256, 49, 3, 2, 1), 35892224), ((2, 23, 21, 14, 512, 87, 3, 1, 1), 29138688),
                         ((2, 159, 141, 83, 11, 64, 3, 2, 1), 252556544), ((2, 31, 20, 16, 119, 192, 3, 1, 1), 31621120)):
        d = mc.make_desc(*args, torch.bfloat16)
        assert mc.workspace_bytes(d, 2) > before >= mc.min_workspace_bytes(d, 2), args
        assert "wgrad_implicit_gemm" in mc.kernel_detail(d, 2, before) and "wgrad_implicit_gemm" not in mc.kernel_detail(d, 2), args
    d = mc.make_desc(1, 16, 16, 32, 1024, 1024, 3, 1, 1, torch.bfloat16)     # three times the time: refused, as before
    assert mc.min_workspace_bytes(d, 2) == mc.workspace_bytes(d, 2)
