"""The GEMM kernels that share the scaled matmul's shapes, at the edges of
their tiles, through the C ABI.

Outputs of few tiles run on the wave kernel (16, 32 or 64 x 64 tiles, K split
over the 4 waves of a workgroup), outputs that 256 x 256 tiles do not spread
over the chip on the 128-row kernel (and some with a fused epilogue), the rest
on the 256 x 256 kernels. Whatever runs: P1 (codes, scale and statistic equal the
oracle's epilogue of the kernel's own accumulator, bit for bit), P2 (the
accumulator against the oracle's fp64 sum), and the dynamic rescale's three
ways (single pass, GEMM + cast kernel, the recovery of a grid that gave up)
give the same bits.

A call needs no kernel that clears its workspace header, and takes its tag
out of it when it is done: replays of a captured graph, with eager calls on
the same workspace in between, equal the eager result.
"""
import itertools
import os

import numpy as np
import pytest
import torch

from paper_2407_17353_amd import binding as sc
from paper_2407_17353_amd import workloads as wl
from tests.gemm_kinds import SHORT_K
from tests.helpers import check_p1, check_p2_full, gpu_matmul, say, stored_with_padding

pytestmark = pytest.mark.gpu
DEV = "cuda"

# M around the tile heights (16, 32, 64, 128), N around 64, 128 and 256
# columns, K around the 128-deep step and the 4 waves' share of it (512)
SHAPES = [(16, 64, 128), (17, 63, 127), (32, 65, 512), (33, 130, 513), (64, 256, 640),
          (65, 257, 1023), (128, 1088, 129), (129, 300, 2049), (700, 1500, 255),
          (1030, 2100, 200), (2050, 4000, 130)]


def _operands(M, N, K, fa, fb, ta, tb, seed):
    A = wl.fp8_normal((M, K), fa, seed, "cpu", 10.0 if fa == sc.E5M2 else None)
    B = wl.fp8_normal((K, N), fb, seed + 1, "cpu", 10.0 if fb == sc.E5M2 else None)
    return (A.t().contiguous() if ta else A), (B.t().contiguous() if tb else B)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("ta,tb", itertools.product((False, True), repeat=2), ids=lambda v: "T" if v else "N")
def test_dynamic_rescale_three_ways(shape, ta, tb, monkeypatch):
    M, N, K = shape
    fa, fb, fout = [(0, 0, 0), (1, 0, 1), (0, 1, 2), (1, 1, 0)][(M + N + K + 2 * ta + tb) % 4]
    say(f"case three ways {shape} ta={ta} tb={tb} fmts={fa},{fb}->{fout}")
    A, B = _operands(M, N, K, fa, fb, ta, tb, 40 + M + N)
    args = (A, fa, ta, -1, B, fb, tb, 2, fout)
    single = gpu_matmul(*args)
    check_p1(*single, K, -1, 2, fout)
    if M * N * K < 3e8:
        check_p2_full(single[3], A, fa, ta, B, fb, tb)
    plain = gpu_matmul(*args, want_acc=False)
    monkeypatch.setenv("SCALIFY_SINGLE_PASS", "0")
    pair = gpu_matmul(*args)
    monkeypatch.setenv("SCALIFY_SINGLE_PASS", "1")
    monkeypatch.setenv("SCALIFY_SPIN_TICKS", "0")
    gave_up = gpu_matmul(*args)
    for other in (plain, pair, gave_up):
        assert np.array_equal(other[0], single[0]) and other[1:3] == single[1:3]
    for other in (pair, gave_up):
        assert np.array_equal(other[3].view(np.uint32), single[3].view(np.uint32))


@pytest.mark.parametrize("shape", [(32, 4096, 512), (256, 1000, 384), (1500, 1024, 256), (2304, 4096, 256)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("mode", [sc.RESCALE_AMAX, sc.RESCALE_DELAYED, sc.RESCALE_NONE])
def test_replays_on_a_shared_workspace(shape, mode):
    """Replays of a captured call carry the same tag; the workspace starts with
    arbitrary contents and serves eager calls of other sizes in between."""
    M, N, K = shape
    say(f"case replays {shape} mode={mode}")
    out = sc.empty_scaled(M, N, sc.E4M3, DEV)
    amax = torch.full((1,), -1.0, device=DEV)
    ws = sc.workspace(sc.scalify_matmul_workspace_size(M, N, sc.E4M3, sc.RESCALE_AMAX) + 4096, DEV)
    ws.fill_(0xAB)
    A = [stored_with_padding(wl.fp8_normal((M, K), 0, 7 + i), DEV) for i in range(2)]
    A_in = A[0].clone()
    a = sc.ScaledArray(A_in, 0, sc.scale_tensor(1, DEV))
    b = sc.ScaledArray(stored_with_padding(wl.fp8_normal((K, N), 0, 9), DEV), 0, sc.scale_tensor(-2, DEV))
    kw = {"rescale": mode, "amax_out": amax, "ws": ws}
    if mode == sc.RESCALE_DELAYED:
        kw["amax_in"] = torch.full((1,), 3.0, device=DEV)

    def eager(x):
        o, am = sc.empty_scaled(M, N, sc.E4M3, DEV), torch.zeros(1, device=DEV)
        sc.scalify_matmul(sc.ScaledArray(x, 0, a.scale), b, o, **{**kw, "amax_out": am})
        torch.cuda.synchronize()
        return o.data.clone(), o.scale.item(), am.item()

    want = [eager(x) for x in A]
    g = torch.cuda.CUDAGraph()
    sc.scalify_matmul(a, b, out, **kw)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        sc.scalify_matmul(a, b, out, **kw)
    small = sc.empty_scaled(48, 80, sc.E4M3, DEV)
    sa = sc.ScaledArray(A[0][:48].clone() if M >= 48 else A[0][:M], 0, None)
    for i in range(6):
        A_in.copy_(A[i % 2])
        out.data.zero_()
        amax.fill_(-1.0)
        g.replay()
        if i % 3 == 2:
            g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.data, want[i % 2][0])
        assert out.scale.item() == want[i % 2][1] and amax.item() == want[i % 2][2]
        if M >= 48 and N >= 80:  # an eager call of another size on the same workspace
            sc.scalify_matmul(sa, sc.ScaledArray(b.data[:, :80], 0, None), small, rescale=sc.RESCALE_AMAX, ws=ws)


@pytest.mark.parametrize("mode", [sc.RESCALE_DELAYED, sc.RESCALE_NONE])
@pytest.mark.parametrize("shape", [(40, 4000, 256), (1500, 1024, 384)], ids=lambda s: "x".join(map(str, s)))
def test_output_scale_may_be_an_input_scale(mode, shape):
    """The output scale shares memory with an input scale (and the statistic
    with amax_in): written only once every workgroup has read it."""
    M, N, K = shape
    say(f"case aliased scales {shape} mode={mode}")
    a = sc.ScaledArray(stored_with_padding(wl.fp8_normal((M, K), 0, 3), DEV), 0, sc.scale_tensor(4, DEV))
    b = sc.ScaledArray(stored_with_padding(wl.fp8_normal((K, N), 0, 4), DEV), 0, sc.scale_tensor(-3, DEV))
    res = []
    for alias in (False, True):
        s = sc.scale_tensor(4, DEV)
        stat = torch.full((1,), 3.0, device=DEV)
        o = sc.empty_scaled(M, N, sc.E4M3, DEV)
        out = sc.ScaledArray(o.data, sc.E4M3, s if alias else o.scale)
        kw = {}
        if mode == sc.RESCALE_DELAYED:
            kw = {"amax_in": stat, "amax_out": stat if alias else torch.zeros(1, device=DEV)}
        sc.scalify_matmul(sc.ScaledArray(a.data, 0, s), b, out, rescale=mode, **kw)
        torch.cuda.synchronize()
        res.append((out.data.clone(), out.scale.item(), kw.get("amax_out", stat).item()))
    assert torch.equal(res[0][0], res[1][0]) and res[0][1:] == res[1][1:]


@pytest.mark.parametrize("mode", [sc.RESCALE_AMAX, sc.RESCALE_NONE])
@pytest.mark.parametrize("shape", [(40, 4096, 300), (1536, 4096, 130), (512, 4096, 4100), (2040, 4096, 4100),
                                   (3000, 4096, 130), (3001, 8200, 130), (2048, 16384, 40), (513, 70000, 16)],
                         ids=lambda s: "x".join(map(str, s)))
def test_fused_epilogue_that_fuses_nothing(shape, mode):
    """A call with a fused epilogue that changes nothing (the pre-cast value is
    exported) may run on another kernel than the plain call: the same bits."""
    M, N, K = shape
    say(f"case fused nothing {shape} mode={mode}")
    a = sc.ScaledArray(stored_with_padding(wl.fp8_normal((M, K), 0, 3), DEV), 0, sc.scale_tensor(2, DEV))
    b = sc.ScaledArray(stored_with_padding(wl.fp8_normal((K, N), 0, 4), DEV), 0, sc.scale_tensor(-3, DEV))
    res = []
    for pre in (None, torch.empty((M, N), device=DEV)):
        out, amax = sc.empty_scaled(M, N, sc.E4M3, DEV), torch.zeros(1, device=DEV)
        sc.scalify_matmul(a, b, out, rescale=mode, amax_out=amax, pre_out=pre)
        torch.cuda.synchronize()
        res.append((out.data.clone(), out.scale.item(), amax.item()))
    assert torch.equal(res[0][0], res[1][0]) and res[0][1:] == res[1][1:]


@pytest.mark.parametrize("shape", [(2100, 4100, 900), (4200, 4200, 900), (1100, 4000, 4500), *SHORT_K],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("ta,tb", [(False, False), (True, True)], ids=["NN", "TT"])
def test_modes_and_epilogues_sum_in_one_order(shape, ta, tb):
    """A call may take another kernel with a statistic than without one, and
    another with a fused epilogue: the accumulators are the same bits."""
    M, N, K = shape
    say(f"case one order {shape} ta={ta} tb={tb}")
    A, B = _operands(M, N, K, 0, 1, ta, tb, 60)
    a = sc.ScaledArray(stored_with_padding(A, DEV), 0, sc.scale_tensor(2, DEV), ta)
    b = sc.ScaledArray(stored_with_padding(B, DEV), 1, sc.scale_tensor(-3, DEV), tb)
    accs = []
    for kw in ({"rescale": sc.RESCALE_AMAX}, {"rescale": sc.RESCALE_NONE},
               {"rescale": sc.RESCALE_NONE, "amax_out": torch.zeros(1, device=DEV)},
               {"rescale": sc.RESCALE_AMAX, "activation": sc.ACT_RELU}):
        acc = torch.empty((M, N), device=DEV)
        sc.scalify_matmul(a, b, sc.empty_scaled(M, N, sc.E4M3, DEV), acc_out=acc, **kw)
        torch.cuda.synchronize()
        accs.append(acc.view(torch.int32))
    assert all(torch.equal(accs[0], x) for x in accs[1:])
