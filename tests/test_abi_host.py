"""Host-side checks of the C ABI (no GPU needed): the library loads, exports
every entry point declared in include/scalify.h, computes the scale rule and
workspace sizes, and rejects bad arguments with the documented status before
any launch (the pointers below are never dereferenced)."""
import ctypes
import os
import re
import subprocess

import pytest

from oracle import oracle as orc
from paper_2407_17353_amd import binding as sc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "scalify.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(scalify_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_function():
    lib = sc.load_library()
    names = declared_functions()
    assert set(names) == set(sc.EXPORTED), names
    for name in names:
        assert hasattr(lib, name), name


def test_the_entry_points_draw_on_nothing_that_throws():
    """C callers cannot catch: the per-call tag comes from the clock, not from
    std::random_device, whose constructor and calls may throw."""
    out = subprocess.run(["nm", "-D", "--undefined-only", sc.LIB_PATH], capture_output=True, text=True, check=True)
    assert "random_device" not in out.stdout


def test_writable_state_of_the_library():
    """Every object that the library's host code may write between calls is one
    of these, all safe with several threads and devices: the CU counts
    (atomics, by device), the next tag (an atomic), and the scratch addresses
    under their mutex."""
    out = subprocess.run(["nm", "-C", sc.LIB_PATH], capture_output=True, text=True, check=True).stdout
    objects = re.findall(r"^\S+ [bBdD] (.*)$", out, flags=re.M)
    mine = [o for o in objects if re.search(r"scalify::|\(anonymous namespace\)", o)
            and not o.endswith(")") and not o.startswith("guard variable")]  # (not the kernels' handles)
    # (scratch: the host's stand-in for the device array of that name, never read)
    assert sorted(o.split("::")[-1] for o in mine) == ["cus", "g_scratch_mutex", "g_scratch_ptr", "next", "scratch"], mine


def test_scale_rule_matches_oracle():
    for K in list(range(0, 3000)) + [8192, 11008, 12288, 16384, 1 << 40]:
        expect = orc.matmul_scale_log2(K) if K > 0 else 0
        assert sc.scalify_matmul_scale_log2(K) == expect, K


def test_workspace_sizes():
    assert sc.scalify_matmul_workspace_size(8192, 8192, sc.E4M3) == 256 + 8192 * 8192 * 2
    assert sc.scalify_matmul_workspace_size(17, 33, sc.E5M2) == 256 + 17 * 48 * 2
    assert sc.scalify_matmul_workspace_size(10, 10, sc.F16) == 256 + 10 * 16 * 4
    assert sc.scalify_matmul_workspace_size(10, 10, sc.F32) == 0      # not an output type
    assert sc.scalify_matmul_workspace_size(-1, 10, sc.E4M3) == 0
    # the delayed rescale casts inside the GEMM: header only
    assert sc.scalify_matmul_workspace_size(8192, 8192, sc.E4M3, sc.RESCALE_DELAYED) == 256
    assert sc.scalify_matmul_workspace_size(10, 10, sc.F16, sc.RESCALE_DELAYED) == 256
    assert sc.scalify_matmul_workspace_size(10, 10, sc.E4M3, 3) == 0
    assert sc.scalify_rescale_workspace_size(123) == 256


def test_status_strings():
    lib = sc.load_library()
    for code in range(9):
        assert lib.scalify_status_string(code)
    assert lib.scalify_status_string(99) == b"unknown status"


FAKE = 0x10000000  # 16-byte aligned, never dereferenced: every case fails validation first


def arr(rows, cols, dtype=sc.E4M3, ld=None, trans=0, data=FAKE, scale=FAKE + 4096):
    if ld is None:
        ld = max(16, ((rows if trans else cols) + 15) // 16 * 16)
    return sc.CScaledArray(data, scale, dtype, trans, rows, cols, ld)


def call_matmul(a, b, out, opts=None, ws=FAKE + 8192, ws_bytes=1 << 40):
    if opts is None:
        opts = sc.CMatmulOpts(out.dtype, sc.RESCALE_AMAX, 0, 1, None, None, None)
    lib = sc.load_library()
    return lib.scalify_matmul(ctypes.byref(a), ctypes.byref(b), ctypes.byref(out),
                              ctypes.byref(opts), ws, ws_bytes, None)


@pytest.mark.parametrize("case,status", [
    ("null_scale_out", 1), ("bad_a_dtype", 2), ("f32_b", 2), ("out_dtype_mismatch", 2),
    ("bad_mode", 7), ("delayed_without_statistic", 1), ("bad_target", 7), ("out_trans", 4), ("k_mismatch", 3), ("n_mismatch", 3),
    ("negative", 3), ("ld_small", 3), ("ld_unaligned", 5), ("ptr_unaligned", 5),
    ("ws_small", 6), ("ws_null", 6), ("ws_unaligned", 6), ("null_data", 1), ("too_big", 3),
    ("channel_b_unaligned", 5), ("channel_a_unaligned", 5),
    ("mx_a_only", 1), ("mx_b_only", 1), ("mx_unaligned", 5), ("mx_with_activation", 7),
    ("mx_with_channel", 7),
])
def test_matmul_argument_errors(case, status):
    a, b, out = arr(64, 128), arr(128, 32), arr(64, 32)
    kw = {}
    if case == "null_scale_out":
        out = arr(64, 32, scale=None)
    elif case == "bad_a_dtype":
        a = arr(64, 128, dtype=sc.F16)
    elif case == "f32_b":
        b = arr(128, 32, dtype=sc.F32)
    elif case == "out_dtype_mismatch":
        kw["opts"] = sc.CMatmulOpts(sc.E5M2, 1, 0, 1, None, None, None)
    elif case == "bad_mode":
        kw["opts"] = sc.CMatmulOpts(sc.E4M3, 3, 0, 1, None, None, None)
    elif case == "delayed_without_statistic":
        kw["opts"] = sc.CMatmulOpts(sc.E4M3, sc.RESCALE_DELAYED, 0, 1, None, None, None, None)
    elif case == "bad_target":
        kw["opts"] = sc.CMatmulOpts(sc.E4M3, 1, 5000, 1, None, None, None)
    elif case == "out_trans":
        out = arr(64, 32, trans=1)
    elif case == "k_mismatch":
        b = arr(127, 32)
    elif case == "n_mismatch":
        out = arr(64, 31)
    elif case == "negative":
        a = arr(-1, 128)
    elif case == "ld_small":
        a = arr(64, 128, ld=112)
    elif case == "ld_unaligned":
        a = arr(64, 128, ld=136)
    elif case == "ptr_unaligned":
        b = arr(128, 32, data=FAKE + 8)
    elif case == "ws_small":
        kw["ws_bytes"] = 256
    elif case == "ws_null":
        kw["ws"] = None
    elif case == "ws_unaligned":
        kw["ws"] = FAKE + 16
    elif case == "null_data":
        a = arr(64, 128, data=None)
    elif case == "too_big":
        a, b, out = arr(1 << 17, 1 << 15), arr(1 << 15, 32), arr(1 << 17, 32)
    elif case == "channel_b_unaligned":
        o = sc.CMatmulOpts(sc.E4M3, 1, 0, 1)
        o.b_channel_scale = FAKE + 20
        kw["opts"] = o
    elif case == "channel_a_unaligned":
        o = sc.CMatmulOpts(sc.E4M3, 1, 0, 1)
        o.a_channel_scale = FAKE + 2
        kw["opts"] = o
    elif case.startswith("mx_"):
        o = sc.CMatmulOpts(sc.E4M3, 1, 0, 1)
        o.a_block_scale = None if case == "mx_b_only" else FAKE + 65536
        o.b_block_scale = None if case == "mx_a_only" else FAKE + 131072
        if case == "mx_unaligned":
            o.b_block_scale = FAKE + 131072 + 2
        elif case == "mx_with_activation":
            o.activation = sc.ACT_RELU
        elif case == "mx_with_channel":
            o.a_channel_scale = FAKE + 196608
        kw["opts"] = o
    assert call_matmul(a, b, out, **kw) == status


@pytest.mark.parametrize("case,status", [
    ("shape", 3), ("trans", 4), ("strided", 4), ("alias_size", 4), ("out_f32", 2),
    ("null_out_scale", 1), ("unaligned", 5),
])
def test_elementwise_argument_errors(case, status):
    lib = sc.load_library()
    x, y = arr(8, 64, dtype=sc.F32, ld=64), arr(8, 64, ld=64)
    if case == "shape":
        y = arr(8, 63, ld=63)
    elif case == "trans":
        y = arr(8, 64, ld=8, trans=1)
    elif case == "strided":
        x = arr(8, 64, dtype=sc.F32, ld=80)
    elif case == "alias_size":
        y = arr(8, 64, ld=64, data=FAKE)       # same buffer, 1-byte vs 4-byte elements
    elif case == "out_f32":
        y = arr(8, 64, dtype=sc.F32, ld=64, data=FAKE + 65536)
    elif case == "null_out_scale":
        y = arr(8, 64, ld=64, data=FAKE + 65536, scale=None)
    elif case == "unaligned":
        y = arr(8, 64, ld=64, data=FAKE + 65536 + 4)
    if case not in ("alias_size",) and y.data == FAKE:
        y.data = FAKE + 65536
    assert lib.scalify_cast(ctypes.byref(x), ctypes.byref(y), 1, None) == status
    assert lib.scalify_rescale(ctypes.byref(x), ctypes.byref(y), 1, 0, 1, FAKE + 131072, 256,
                               None) == status


def test_rescale_and_set_scaling_specific_errors():
    lib = sc.load_library()
    x, y = arr(4, 64, dtype=sc.F32, ld=64), arr(4, 64, ld=64, data=FAKE + 65536)
    assert lib.scalify_rescale(ctypes.byref(x), ctypes.byref(y), 3, 0, 1, FAKE + 131072, 256, None) == 7
    assert lib.scalify_rescale(ctypes.byref(x), ctypes.byref(y), 1, 0, 1, FAKE + 131072, 128, None) == 6
    assert lib.scalify_set_scaling(ctypes.byref(x), ctypes.byref(y), 128, 1, None) == 7
    y2 = arr(4, 64, ld=64, data=FAKE + 65536, scale=x.scale)
    assert lib.scalify_set_scaling(ctypes.byref(x), ctypes.byref(y2), 3, 1, None) == 4


def test_fused_workspace_sizes():
    """A fused residual add / activation / pre_out keeps an fp32 intermediate."""
    assert sc.scalify_matmul_workspace_size_opts(8192, 8192, sc.E4M3) == 256 + 8192 * 8192 * 2
    assert sc.scalify_matmul_workspace_size_opts(8192, 8192, sc.E4M3, fused=True) == \
        256 + 8192 * 8192 * 4
    assert sc.scalify_matmul_workspace_size_opts(17, 33, sc.E5M2, fused=True) == 256 + 17 * 48 * 4
    assert sc.scalify_matmul_workspace_size_opts(10, 10, sc.F16, fused=True) == 256 + 10 * 16 * 4
    assert sc.scalify_matmul_workspace_size_opts(10, 10, sc.E4M3, sc.RESCALE_DELAYED, True) == 256
    # channel scales keep the fp32 intermediate as well
    o = sc.CMatmulOpts(sc.E4M3, sc.RESCALE_AMAX, 0, 1)
    o.b_channel_scale = FAKE
    assert sc.load_library().scalify_matmul_workspace_size_opts(10, 10, ctypes.byref(o)) == 256 + 10 * 16 * 4
    # so do MX block scales
    o = sc.CMatmulOpts(sc.E4M3, sc.RESCALE_AMAX, 0, 1)
    o.a_block_scale, o.b_block_scale = FAKE, FAKE + 4096
    assert sc.load_library().scalify_matmul_workspace_size_opts(10, 10, ctypes.byref(o)) == 256 + 10 * 16 * 4
    assert sc.load_library().scalify_matmul_workspace_size_opts(10, 10, None) == 0


def test_mx_packed_bytes_and_pack_argument_errors():
    """256 bytes per 128-k step and 64-row group; the pack entry point checks
    its arguments before launching anything."""
    for rows, K in ((1, 1), (64, 128), (65, 129), (8192, 8192), (11008, 4096)):
        assert sc.scalify_mx_packed_bytes(rows, K) == 256 * ((K + 127) // 128) * ((rows + 63) // 64)
    assert sc.scalify_mx_packed_bytes(0, 64) == 0 and sc.scalify_mx_packed_bytes(64, 0) == 0
    lib = sc.load_library()
    pack = lib.scalify_mx_pack_block_scales
    assert pack(None, 0, 64, 2, None, None) == 0           # nothing to pack, nothing launched
    assert pack(None, 16, 64, 2, FAKE, None) == 1           # NULL src
    assert pack(FAKE, 16, 64, 1, FAKE + 4096, None) == 3    # src_ld < ceil(K / 32)
    assert pack(FAKE, -1, 64, 2, FAKE + 4096, None) == 3    # negative rows
    assert pack(FAKE, 16, 64, 2, FAKE + 4098, None) == 5    # dst not 4-byte aligned


def fused_opts(residual=None, act=sc.ACT_NONE, pre_out=None, out_dtype=sc.E4M3,
               mode=sc.RESCALE_AMAX):
    o = sc.CMatmulOpts(out_dtype, mode, 0, 1, None, None, None, None, None, act, pre_out)
    if residual is not None:
        o.residual = ctypes.pointer(residual)
    return o


@pytest.mark.parametrize("case,status", [
    ("act_high", 7), ("act_negative", 7), ("res_f32", 2), ("res_rows", 3), ("res_cols", 3),
    ("res_trans", 4), ("res_ld_small", 3), ("res_ld_unaligned", 5), ("res_f16_ld", 5),
    ("res_ptr_unaligned", 5), ("res_null_data", 1), ("res_overlaps_out", 4),
    ("res_same_data_other_ld", 4), ("res_broadcast_over_out", 4), ("ws_too_small_for_fused", 6),
])
def test_matmul_fused_argument_errors(case, status):
    a, b, out = arr(64, 128), arr(128, 32), arr(64, 32, data=FAKE + (1 << 20))
    res = arr(64, 32, data=FAKE + (2 << 20))
    kw = {}
    opts = None
    if case == "act_high":
        opts = fused_opts(act=4)
    elif case == "act_negative":
        opts = fused_opts(act=-1)
    elif case == "res_f32":
        opts = fused_opts(arr(64, 32, dtype=sc.F32, data=FAKE + (2 << 20)))
    elif case == "res_rows":
        opts = fused_opts(arr(63, 32, data=FAKE + (2 << 20)))
    elif case == "res_cols":
        opts = fused_opts(arr(64, 48, data=FAKE + (2 << 20)))
    elif case == "res_trans":
        opts = fused_opts(arr(64, 32, trans=1, data=FAKE + (2 << 20)))
    elif case == "res_ld_small":
        opts = fused_opts(arr(64, 32, ld=16, data=FAKE + (2 << 20)))
    elif case == "res_ld_unaligned":
        opts = fused_opts(arr(64, 32, ld=40, data=FAKE + (2 << 20)))
    elif case == "res_f16_ld":
        opts = fused_opts(arr(64, 32, dtype=sc.F16, ld=36, data=FAKE + (2 << 20)))
    elif case == "res_ptr_unaligned":
        opts = fused_opts(arr(64, 32, data=FAKE + (2 << 20) + 4))
    elif case == "res_null_data":
        opts = fused_opts(arr(64, 32, data=None))
    elif case == "res_overlaps_out":
        opts = fused_opts(arr(64, 32, data=FAKE + (1 << 20) + 64))
    elif case == "res_same_data_other_ld":
        opts = fused_opts(arr(64, 32, ld=48, data=FAKE + (1 << 20)))
    elif case == "res_broadcast_over_out":
        opts = fused_opts(arr(64, 32, ld=0, data=FAKE + (1 << 20)))
    elif case == "ws_too_small_for_fused":
        opts = fused_opts(res)
        kw["ws_bytes"] = sc.scalify_matmul_workspace_size(64, 32, sc.E4M3)
    assert call_matmul(a, b, out, opts=opts, **kw) == status


def _ln_fwd(x, out, gamma=None, beta=None, eps=1e-5, pre=None):
    lib = sc.load_library()
    return lib.scalify_layernorm_fwd(ctypes.byref(x), gamma, beta, eps, ctypes.byref(out), 1, pre, None)


def _ln_bwd(dy, x, dx, mode=sc.RESCALE_AMAX, eps=1e-5, ws=FAKE + 8192, ws_bytes=1 << 40, **kw):
    lib = sc.load_library()
    return lib.scalify_layernorm_bwd(ctypes.byref(dy), ctypes.byref(x), kw.get("gamma"), eps,
                                     ctypes.byref(dx), kw.get("dgamma"), kw.get("dbeta"), mode, 0, 1,
                                     None, kw.get("pre"), ws, ws_bytes, None)


def test_layernorm_workspace_size():
    # header + 4 floats per row + per 32-row tile 2 x round_up(D, 16) floats
    assert sc.scalify_layernorm_bwd_workspace_size(16384, 4096) == 256 + 4 * (4 * 16384 + 512 * 2 * 4096)
    assert sc.scalify_layernorm_bwd_workspace_size(33, 17) == 256 + 4 * (4 * 33 + 2 * 2 * 32)
    assert sc.scalify_layernorm_bwd_workspace_size(0, 16) == 256 + 4 * (1 * 2 * 16)
    assert sc.scalify_layernorm_bwd_workspace_size(10, 8193) == 0


@pytest.mark.parametrize("case,status", [
    ("d_too_big", 3), ("d_zero", 3), ("out_f32", 2), ("shape", 3), ("trans", 4), ("ld_small", 3),
    ("ld_unaligned", 5), ("gamma_unaligned", 5), ("eps_negative", 7), ("eps_nan", 7),
    ("null_scale", 1), ("overlap", 4),
])
def test_layernorm_fwd_argument_errors(case, status):
    x, out = arr(8, 64, dtype=sc.F16, ld=64), arr(8, 64, ld=64, data=FAKE + (1 << 20))
    kw = {}
    if case == "d_too_big":
        x, out = arr(8, 8200, dtype=sc.F16, ld=8200), arr(8, 8200, ld=8208, data=FAKE + (1 << 20))
    elif case == "d_zero":
        x, out = arr(8, 0, dtype=sc.F16, ld=16), arr(8, 0, ld=16, data=FAKE + (1 << 20))
    elif case == "out_f32":
        out = arr(8, 64, dtype=sc.F32, ld=64, data=FAKE + (1 << 20))
    elif case == "shape":
        out = arr(8, 63, ld=64, data=FAKE + (1 << 20))
    elif case == "trans":
        x = arr(8, 64, dtype=sc.F16, ld=8, trans=1)
    elif case == "ld_small":
        x = arr(8, 64, dtype=sc.F16, ld=56)
    elif case == "ld_unaligned":
        x = arr(8, 64, dtype=sc.F16, ld=68)
    elif case == "gamma_unaligned":
        kw["gamma"] = FAKE + (2 << 20) + 4
    elif case == "eps_negative":
        kw["eps"] = -1.0
    elif case == "eps_nan":
        kw["eps"] = float("nan")
    elif case == "null_scale":
        out = arr(8, 64, ld=64, data=FAKE + (1 << 20), scale=None)
    elif case == "overlap":
        out = arr(8, 64, ld=64, data=FAKE + 64)
    assert _ln_fwd(x, out, **kw) == status


@pytest.mark.parametrize("case,status", [
    ("mode", 7), ("shape_dy", 3), ("dx_f32", 2), ("ws_small", 6), ("ws_null", 6),
    ("dgamma_unaligned", 5), ("dx_overlaps_x", 4),
])
def test_layernorm_bwd_argument_errors(case, status):
    dy = arr(8, 64, dtype=sc.E5M2, ld=64)
    x = arr(8, 64, dtype=sc.F16, ld=64, data=FAKE + (1 << 20))
    dx = arr(8, 64, dtype=sc.E5M2, ld=64, data=FAKE + (2 << 20))
    kw = {}
    if case == "mode":
        kw["mode"] = sc.RESCALE_DELAYED
    elif case == "shape_dy":
        dy = arr(9, 64, dtype=sc.E5M2, ld=64)
    elif case == "dx_f32":
        dx = arr(8, 64, dtype=sc.F32, ld=64, data=FAKE + (2 << 20))
    elif case == "ws_small":
        kw["ws_bytes"] = 256
    elif case == "ws_null":
        kw["ws"] = None
    elif case == "dgamma_unaligned":
        kw["dgamma"] = FAKE + (3 << 20) + 8
    elif case == "dx_overlaps_x":
        dx = arr(8, 64, dtype=sc.E5M2, ld=64, data=FAKE + (1 << 20) + 128)
    assert _ln_bwd(dy, x, dx, **kw) == status
