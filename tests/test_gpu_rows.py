"""LayerNorm and rescale at the edges of their kernels' row and block splits,
through the C ABI.

A LayerNorm row belongs to one, two or four waves (2048, 4096 and 8192
columns): the single-read kernels give the bits of the multi-pass ones
(SCALIFY_LN_SINGLE_READ=0) at the widths where that split and the lanes'
chunks can go wrong, rows that do not fill a workgroup included, and the
statistic they report is the maximum of the exported gradient. The rescale and
the LayerNorm backward need no kernel that clears their header: replays of
captured calls, on a workspace with arbitrary contents, equal the eager ones.
"""
import numpy as np
import pytest
import torch

from paper_2407_17353_amd import binding as sc
from tests.helpers import say

pytestmark = pytest.mark.gpu
DEV = "cuda"
TORCH = {sc.E4M3: torch.float8_e4m3fn, sc.E5M2: torch.float8_e5m2, sc.F16: torch.float16, sc.F32: torch.float32}


def _rows(R, D, fmt, seed, scale=None):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randn((R, D), generator=g, device=DEV) + 0.5
    if scale is not None:
        x = x * torch.exp2(-scale * torch.rand((R, 1), generator=g, device=DEV))
    ld = max(16, (D + 15) // 16 * 16)
    st = torch.empty((R, ld), dtype=sc.STORAGE_DTYPE[fmt], device=DEV)
    st.view(torch.uint8).fill_(0x7F)
    st[:, :D] = x.to(TORCH[fmt]).view(st.dtype)
    return sc.ScaledArray(st[:, :D], fmt, sc.scale_tensor(2, DEV))


WIDTHS = [1, 15, 64, 1023, 1024, 1040, 2047, 2048, 2049, 3072, 4095, 4096, 4097, 6144, 6150, 8191, 8192]


@pytest.mark.parametrize("D", WIDTHS)
@pytest.mark.parametrize("fx,fd,fo", [(sc.F16, sc.E5M2, sc.E5M2), (sc.F32, sc.F16, sc.F16), (sc.E4M3, sc.F32, sc.E4M3)],
                         ids=["f16-e5m2", "f32-f16", "e4m3-f32"])
def test_single_read_equals_multi_pass(D, fx, fd, fo, monkeypatch):
    _single_equals_multi(7 if D > 64 else 4100, D, fx, fd, fo, monkeypatch)


# more rows than the grid has places (768 or 1024 workgroups of 1, 2 or 4 rows
# on 256 CUs): the next row's loads and the reuse of the sums' LDS slots, by
# waves per row
@pytest.mark.parametrize("R,D", [(6300, 72), (6200, 2048), (3200, 2049), (3100, 4096), (1700, 4100), (1600, 8192)])
@pytest.mark.parametrize("fx,fd,fo", [(sc.F16, sc.E5M2, sc.E5M2), (sc.F32, sc.F16, sc.F16)], ids=["f16-e5m2", "f32-f16"])
def test_single_read_equals_multi_pass_over_many_rows(R, D, fx, fd, fo, monkeypatch):
    for peak in (0, R - 2):  # the largest gradient among the first rows and the last
        _single_equals_multi(R, D, fx, fd, fo, monkeypatch, peak)


def _single_equals_multi(R, D, fx, fd, fo, monkeypatch, peak=None):
    say(f"case layernorm rows R={R} D={D} fmts={fx},{fd}->{fo} peak={peak}")
    x, dy = _rows(R, D, fx, D), _rows(R, D, fd, D + 1, 10.0)
    if peak is not None:
        dy.data[peak, D // 3] = torch.tensor([1000.0], device=DEV).to(TORCH[fd]).view(dy.data.dtype)[0]
    gamma = 1.0 + 0.1 * torch.randn(D, device=DEV)
    beta = 0.1 * torch.randn(D, device=DEV)
    res = []
    for single in ("1", "0"):
        monkeypatch.setenv("SCALIFY_LN_SINGLE_READ", single)
        y, dx = sc.empty_scaled(R, D, fo, DEV), sc.empty_scaled(R, D, fo, DEV)
        pre, pre_b = torch.zeros((R, D), device=DEV), torch.zeros((R, D), device=DEV)
        dg, db, am = torch.zeros(D, device=DEV), torch.zeros(D, device=DEV), torch.zeros(1, device=DEV)
        ws = sc.workspace(sc.scalify_layernorm_bwd_workspace_size(R, D), DEV)
        ws.fill_(0xAB)
        sc.scalify_layernorm_fwd(x, y, gamma=gamma, beta=beta, pre_out=pre)
        sc.scalify_layernorm_bwd(dy, x, dx, gamma=gamma, dgamma=dg, dbeta=db, amax_out=am, pre_out=pre_b, ws=ws)
        torch.cuda.synchronize()
        assert am.item() == pre_b.abs().max().item()
        assert peak is None or am.item() == pre_b[peak].abs().max().item()
        res.append([t.contiguous().view(torch.uint8).cpu().numpy()
                    for t in (y.data, pre, dx.data, dx.scale, pre_b, dg, db, am)])
    for a, b in zip(*res):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [1, 1023, 1024, 5 * 1024 + 7, 2048 * 1024 + 3, 3 << 22])
@pytest.mark.parametrize("mode", [sc.RESCALE_AMAX, sc.RESCALE_NONE])
def test_rescale_replays_on_a_dirty_workspace(n, mode):
    say(f"case rescale replays n={n} mode={mode}")
    x = [torch.randn((1, n), device=DEV) * 2.0 ** (5 * i) for i in range(2)]
    x_in = x[0].clone()
    out = sc.ScaledArray(torch.empty((1, n), dtype=torch.uint8, device=DEV), sc.E4M3, torch.empty(1, device=DEV))
    ws = sc.workspace(256, DEV)
    ws.fill_(0xAB)
    arr = sc.ScaledArray(x_in, sc.F32, sc.scale_tensor(3, DEV))
    want = []
    for t in x:
        sc.scalify_rescale(sc.ScaledArray(t, sc.F32, arr.scale), out, mode=mode, ws=ws)
        torch.cuda.synchronize()
        want.append((out.data.clone(), out.scale.item()))
        e = int(np.floor(np.log2(t.abs().max().item()))) if mode == sc.RESCALE_AMAX else 0
        assert out.scale.item() == 2.0 ** (3 + e)
        ref = (t * 2.0 ** -e).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
        assert torch.equal(out.data, ref)
    # the output scale in the input scale's place
    s = sc.scale_tensor(3, DEV)
    sc.scalify_rescale(sc.ScaledArray(x[1], sc.F32, s), sc.ScaledArray(out.data, sc.E4M3, s), mode=mode, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(out.data, want[1][0]) and s.item() == want[1][1]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sc.scalify_rescale(arr, out, mode=mode, ws=ws)
    for i in range(5):
        x_in.copy_(x[i % 2])
        out.data.zero_()
        g.replay()
        if i == 2:
            g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.data, want[i % 2][0]) and out.scale.item() == want[i % 2][1]


def test_layernorm_backward_replays():
    say("case layernorm backward replays")
    R, D = 300, 2512
    x = [_rows(R, D, sc.F16, 3 + i) for i in range(2)]
    x_in = sc.ScaledArray(x[0].data.clone(), sc.F16, x[0].scale)
    dy = _rows(R, D, sc.E5M2, 9, 10.0)
    ws = sc.workspace(sc.scalify_layernorm_bwd_workspace_size(R, D), DEV)
    ws.fill_(0xAB)
    dx = sc.empty_scaled(R, D, sc.E5M2, DEV)
    dg, db = torch.zeros(D, device=DEV), torch.zeros(D, device=DEV)

    def call(a):
        sc.scalify_layernorm_bwd(dy, a, dx, dgamma=dg, dbeta=db, ws=ws)

    want = []
    for a in x:
        call(a)
        torch.cuda.synchronize()
        want.append([t.clone() for t in (dx.data, dx.scale, dg, db)])
    x_in.data.copy_(x[0].data)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(x_in)
    for i in range(5):
        x_in.data.copy_(x[i % 2].data)
        for t in (dx.scale, dg, db):
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        for got, ref in zip((dx.data, dx.scale, dg, db), want[i % 2]):
            assert torch.equal(got, ref)


@pytest.mark.parametrize("D", [1, 100, 8192, 8193, 20000])
@pytest.mark.parametrize("mode", [sc.RESCALE_AMAX, sc.RESCALE_NONE])
def test_layernorm_backward_without_rows(D, mode):
    """R = 0: the scale of the rule, a statistic and parameter gradients of 0;
    nothing is written outside the workspace, which at D > 8192 has no bytes."""
    say(f"case layernorm backward R=0 D={D} mode={mode}")
    need = sc.scalify_layernorm_bwd_workspace_size(0, D)
    assert (need == 0) == (D > 8192)
    buf = torch.full((need + (1 << 20),), 0xAB, dtype=torch.uint8, device=DEV)
    assert buf.data_ptr() % 256 == 0
    empty = lambda fmt, e: sc.ScaledArray(torch.empty((0, D), dtype=sc.STORAGE_DTYPE[fmt], device=DEV), fmt,
                                          sc.scale_tensor(e, DEV))
    dx = empty(sc.E5M2, 0)
    dg, db, am = (torch.full((n,), 7.0, device=DEV) for n in (D, D, 1))
    sc.scalify_layernorm_bwd(empty(sc.E5M2, 5), empty(sc.F16, 2), dx, rescale=mode, dgamma=dg, dbeta=db,
                             amax_out=am, ws=buf)
    torch.cuda.synchronize()
    assert dx.scale.item() == 2.0 ** 3 and am.item() == 0.0
    assert not dg.any() and not db.any()
    assert bool((buf[need:] == 0xAB).all())
