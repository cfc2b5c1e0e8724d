"""GPU parity of the gather kernels (patch rows gathered by LDS DMA) against the
oracle, at the sizes where their index arithmetic has its edges: the plan query
shows that each case takes them."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_close, dev, host, rounded
from paper_1802_04647_amd import dmlnn
from paper_1802_04647_amd.inputs import ConvShape, random_conv_case

pytestmark = pytest.mark.gpu

DT = {"f64": torch.float64, "f32": torch.float32}

CASES = [
    ConvShape(9, 7, 9, 7, 33, 3, 3, 1, 1),      # tiles across images, k tail inside a 16-byte piece
    ConvShape(6, 45, 11, 13, 70, 3, 3, 2, 1),   # four phases of 4, 2, 2 and 1 taps; five-block rows
    ConvShape(5, 5, 17, 15, 20, 5, 5, 3, 2),    # nine phases, uncovered border cells
    ConvShape(7, 6, 13, 13, 18, 2, 3, 4, 0),    # stride above the filter: phases without a tap
    ConvShape(8, 37, 8, 8, 130, 1, 1, 1, 0),    # 1x1: whole planes (16-byte patch rows)
    ConvShape(8, 33, 9, 9, 17, 1, 1, 2, 0),     # 1x1, stride 2: three phases of zeros
    ConvShape(4, 3, 10, 12, 16, 3, 3, 1, 4),    # pad above the filter: cells of padding only
    ConvShape(5, 12, 8, 8, 48, 7, 5, 1, 3),     # 35 taps, non-square
    ConvShape(300, 2, 1, 1, 8, 3, 3, 1, 1),     # one-pixel images: a tile spans 64 of them
    ConvShape(2, 130, 31, 29, 144, 3, 3, 1, 1), # wide tiles, many chunks
]


def _args(s):
    return (s.C, s.Hin, s.Win, s.Hf, s.Wf, s.stride, s.pad)


def test_cases_take_the_gather_kernels():
    seen = set()
    for s in CASES:
        for dt in DT.values():
            for pname in ("forward", "backward_filter", "backward_data"):
                p = dmlnn.conv2d_plan(dt, pname, *s.args())
                seen.add((pname, p["kernel"], p["row_staged"] if "filter" not in pname else p["slice_vec"]))
    for pname in ("forward", "backward_data"):
        assert {(pname, "gather", nt) for nt in (0, 1, 9)} <= seen
    assert {("backward_filter", "wgrad_gather", m) for m in (0, 1, 2)} <= seen


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("s", CASES, ids=str)
def test_gather_parity(s, dt):
    X0, W0, b0, dout0 = random_conv_case(300, s, zero_frac=0.3)
    X, W, b, dout = (rounded(v, dt) for v in (X0, W0, b0, dout0))
    mask = rounded(np.maximum(random_conv_case(301, s)[3], 0.0), dt)
    a = _args(s)
    print(f"\n[gpu] gather {s} {dt}", flush=True)
    out, _, _ = dmlnn.conv2d_forward(dev(X, dt), dev(W, dt), dev(b, dt), *a, relu=False)
    dd, dm = dev(dout, dt), dev(mask, dt)
    dX = dmlnn.conv2d_backward_data(dev(W, dt), dd, dm, *a)
    g = torch.full_like(dd, float("nan"))
    dW, db = dmlnn.conv2d_backward_filter(dev(X, dt), dd, dm, *a, s.F, g_out=g)
    dX1 = dmlnn.conv2d_backward_data(dev(W, dt), g, None, *a)
    dW1, db1 = dmlnn.conv2d_backward_filter(dev(X, dt), g, None, *a, s.F)
    torch.cuda.synchronize()
    assert torch.equal(g, torch.where(dm > 0, dd, torch.zeros_like(dd)))
    for u, v in ((dX, dX1), (dW, dW1), (db, db1)):  # who applies the mask changes nothing
        assert torch.equal(u, v)
    ref_out, _, _ = oracle.conv2d_forward(X, W, b, *a, relu=False)
    ref_dW, ref_db = oracle.conv2d_backward_filter(X, dout, mask, *a, s.F)
    ref_dX = oracle.conv2d_backward_data(W, dout, mask, *a)
    for got, ref, what in ((out, ref_out, "forward"), (dW, ref_dW, "dW"), (db, ref_db, "db"),
                           (dX, ref_dX, "dX")):
        assert_close(host(got), ref, dt, what)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_one_row_of_infinities_stays_in_its_row(dt):
    """The last k-chunk of a filter row fetches the head of the next row: a
    non-finite filter must not reach its neighbour's outputs, nor an image the
    next image's."""
    s = ConvShape(6, 7, 9, 9, 40, 3, 3, 1, 1)
    X, W, b, dout = (dev(rounded(v, dt), dt) for v in random_conv_case(302, s))
    a = _args(s)
    ref, _, _ = dmlnn.conv2d_forward(X, W, b, *a, relu=False)
    Wi, Xn = W.clone(), X.clone()
    Wi[7] = float("inf")
    Xn[2] = float("nan")
    got, _, _ = dmlnn.conv2d_forward(Xn, Wi, b, *a, relu=False)
    dX0 = dmlnn.conv2d_backward_data(W, dout, None, *a)
    gn = dout.clone()
    gn[3] = float("inf")
    dX1 = dmlnn.conv2d_backward_data(W, gn, None, *a)
    torch.cuda.synchronize()
    v, r = got.view(s.N, s.F, -1), ref.view(s.N, s.F, -1)
    rows = [f for f in range(s.F) if f != 7]
    imgs = [n for n in range(s.N) if n != 2]
    assert torch.equal(v[imgs][:, rows], r[imgs][:, rows])
    assert not torch.isfinite(v[2]).any() and not torch.isfinite(v[:, 7]).any()
    keep = [n for n in range(s.N) if n != 3]
    assert torch.equal(dX1[keep], dX0[keep])


@pytest.mark.parametrize("W", [40, 41, 43, 44, 47, 54])
def test_ring_rows_that_end_inside_a_round(W):
    """The fp32 ring's rounds of eight pixels, against a float64 product of the patches."""
    N, C, H, F = 64, 64, 64, 64
    a = (C, H, W, 3, 3, 1, 1)
    plan = dmlnn.conv2d_plan(torch.float32, "backward_filter", N, C, H, W, F, 3, 3, 1, 1)
    assert plan["kernel"] == "wgrad_ring" and plan["row_staged"] & 4, plan
    print(f"\n[gpu] ring W={W}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    X = torch.randn(N, C * H * W, generator=gen, device="cuda")
    g = torch.randn(N, F * H * W, generator=gen, device="cuda")
    dW, db = dmlnn.conv2d_backward_filter(X, g, None, *a, F)[:2]
    cols = torch.nn.functional.unfold(X.double().view(N, C, H, W), 3, padding=1)
    cols = cols.permute(0, 2, 1).reshape(N * H * W, C * 9)
    gm = g.double().view(N, F, H * W).permute(1, 0, 2).reshape(F, N * H * W)
    assert_close(host(dW), host(gm @ cols), "f32", "dW")
    assert_close(host(db), host(gm.sum(1)), "f32", "db")
