"""The fused epilogue (scaled add, activation, channel scales) in every GEMM
kernel that large outputs take, through the C ABI against the CPU oracle: the
sizes of tests/gemm_kinds.py, ragged in M, N and K, each with every residual
format, a bias, every activation and channel scales, in rotating layouts and
formats.

F1 and F2 (tests/test_gpu_fused.py) for the dynamic rescale; its other ways
(GEMM + cast kernel, the recovery of a grid that gave up) and the delayed and
absent rescale have the same pre-cast values bit for bit, and F2 of their own.
"""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2407_17353_amd import binding as sc
from tests.gemm_kinds import FUSED
from tests.helpers import check_p2_sampled, say
from tests.test_gpu_channel import _channels
from tests.test_gpu_fused import ACTS, LAYOUTS, _codes, _oracle_res, _residual_codes, _run, check_fused

pytestmark = pytest.mark.gpu

# (activation, residual format or None, bias, channel scales of)
COMBOS = [("gelu", sc.F16, True, None), ("none", sc.E4M3, False, None), ("relu", sc.E5M2, False, None),
          ("silu", sc.F16, False, None), ("none", None, False, "both"), ("relu", None, False, None),
          ("gelu", sc.E4M3, False, "a"), ("silu", sc.E5M2, True, "b")]


def _finish(run, sa, sb, res, mode, amax_in, fout, sat=True):
    """F2 alone: codes, scale and statistic from the call's own pre-cast values."""
    codes, e_out, amax, _, pre, K = run
    e_c = orc.matmul_scale_log2(K)
    e_w = sa + sb if res is None else max(sa + sb + e_c, res[2])
    ref, e_ref, am_ref = orc.finish_pre(pre, e_w, e_c if res is None else 0, mode, 0, amax_in, sat, fout)
    assert e_out == e_ref and np.float32(amax) == np.float32(am_ref), (e_out, e_ref, amax, am_ref)
    bad = np.count_nonzero(codes.ravel() != ref.ravel())
    assert bad == 0, f"F2: {bad} codes differ"


@pytest.mark.parametrize("combo", COMBOS, ids=lambda c: "-".join(str(v) for v in c))
@pytest.mark.parametrize("kernel", list(FUSED))
def test_fused_epilogues_of_the_large_kernels(kernel, combo, monkeypatch):
    act_name, rfmt, bias, which = combo
    act = ACTS[act_name]
    M, N, K = FUSED[kernel]
    i = COMBOS.index(combo) + 3 * list(FUSED).index(kernel)
    ta, tb = LAYOUTS[(i + i // 4) % 4]
    fa, fb = [(0, 0), (1, 0), (0, 1), (1, 1)][i % 4]
    fout = [sc.E4M3, sc.F16, sc.E5M2][i % 3]
    sa, sb, q = -2, 1, [3, -4, 0, 7][i % 4]
    say(f"case fused {kernel} {combo} {M}x{N}x{K} ta={ta} tb={tb} fmts={fa},{fb}->{fout}")
    A = _codes((K, M) if ta else (M, K), fa, 500 + i, heavy=fa == sc.E5M2)
    B = _codes((N, K) if tb else (K, N), fb, 600 + i, heavy=fb == sc.E5M2)
    res = None
    if rfmt is not None:
        res = (_residual_codes(M, N, rfmt, 700 + i, rows=1 if bias else None, spread=4), rfmt, q)
    ca, cb = _channels(M, N, 800 + i, which=which) if which else (None, None)
    kw = dict(res=res, act=act, ch_a=ca, ch_b=cb)
    args = (A, fa, ta, sa, B, fb, tb, sb, fout)
    run = _run(*args, **kw)
    check_fused(run, sa, sb, fout, res, act, sc.RESCALE_AMAX, ch_a=ca, ch_b=cb)
    check_p2_sampled(run[3], A, fa, ta, B, fb, tb, n_samples=2048)
    for mode, amax_in in ((sc.RESCALE_DELAYED, 5.0), (sc.RESCALE_NONE, 0.0)):
        other = _run(*args, mode=mode, amax_in=amax_in, **kw)
        assert np.array_equal(other[4].view(np.uint32), run[4].view(np.uint32))
        _finish(other, sa, sb, res, mode, amax_in, fout)
    for env in ({"SCALIFY_SINGLE_PASS": "0"}, {"SCALIFY_SINGLE_PASS": "1", "SCALIFY_SPIN_TICKS": "0"}):
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        other = _run(*args, **kw)
        assert np.array_equal(other[0], run[0]) and other[1:3] == run[1:3]
        assert np.array_equal(other[4].view(np.uint32), run[4].view(np.uint32))


@pytest.mark.parametrize("mode", [sc.RESCALE_AMAX, sc.RESCALE_DELAYED])
@pytest.mark.parametrize("kernel", list(FUSED))
def test_fused_residual_in_place_and_specials(kernel, mode):
    """The residual is the output matrix itself, without the export of w; NaN and Inf residual codes, a NaN accumulator
    row; saturating and not."""
    M, N, K = FUSED[kernel]
    i = list(FUSED).index(kernel)
    ta, tb = LAYOUTS[(i + 1) % 4]
    say(f"case fused in place {kernel} {M}x{N}x{K} mode={mode} ta={ta} tb={tb}")
    A = _codes((K, M) if ta else (M, K), sc.E5M2, 41 + i, heavy=True).numpy().copy()
    A[(9, 5) if ta else (5, 9)] = 0x7F  # NaN: row 5 of the product
    A = torch.from_numpy(A)
    B = _codes((N, K) if tb else (K, N), sc.E4M3, 42 + i)
    r = _residual_codes(M, N, sc.E5M2, 43 + i)
    r[M - 1, :8] = [0x7C, 0xFC, 0x7D, 0xFE, 0x00, 0x80, 0x7B, 0xFB]  # +-Inf, NaNs, +-0, +-max
    r[200, 300] = 0x7C
    res = (r, sc.E5M2, -3)
    for sat in (True, False):
        kw = dict(res=res, act=sc.ACT_SILU, mode=mode, amax_in=1.0, sat=sat)
        run = _run(A, sc.E5M2, ta, 0, B, sc.E4M3, tb, 0, sc.E5M2, **kw)
        check_fused(run, 0, 0, sc.E5M2, res, sc.ACT_SILU, mode, amax_in=1.0, sat=sat)
        inp = _run(A, sc.E5M2, ta, 0, B, sc.E4M3, tb, 0, sc.E5M2, inplace=True, want_pre=False, **kw)
        assert np.array_equal(inp[0], run[0]) and inp[1] == run[1]
        assert np.float32(inp[2]) == np.float32(run[2]) or (math.isnan(inp[2]) and math.isnan(run[2]))
