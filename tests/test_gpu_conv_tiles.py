"""GPU parity of the LDS-tiled convolution kernels at the edges of their tiles:
rows and columns one short of, equal to and one past a tile, channel counts
that are padded to the matrix instruction's 16, upsampled inputs at both
strides, one-voxel extents.  Same operands and tolerance as the other
convolution tests (bf16 operands, fp32 sums, against the FP64 oracle)."""
import pytest
import torch

import oracle
from paper_2509_25044_amd import ops
from parity_util import assert_grad
from test_gpu_conv import DEV, SLOPE, _bf, _case

pytestmark = pytest.mark.gpu

# N, Di, Hi, Wi, Ca, Cb, Cout, stride, ups
CASES = [
    (1, 3, 7, 31, 16, 0, 16, 1, False),
    (1, 2, 8, 32, 12, 8, 20, 1, False),
    (2, 1, 9, 33, 4, 0, 16, 1, False),
    (1, 18, 1, 1, 16, 0, 4, 1, False),
    (1, 6, 10, 18, 32, 16, 48, 1, True),
    (1, 2, 18, 34, 20, 4, 16, 1, True),
    (1, 1, 4, 31, 16, 0, 32, 2, False),
    (1, 5, 9, 65, 8, 4, 36, 2, False),
    (1, 6, 10, 66, 32, 16, 16, 2, True),
    (2, 9, 17, 34, 4, 0, 4, 2, False),
]


@pytest.mark.parametrize("case", CASES)
def test_weight_gradient(case):
    print(f"[conv wgrad tiles {case}]", flush=True)
    N, Di, Hi, Wi, Ca, Cb, Cout, s, ups = case
    xa, xb, w, b, geom = _case(*case, seed=3)
    oshape = (N,) + ops.conv_out_shape(geom) + (Cout,)
    g = torch.Generator().manual_seed(4)
    dy, y = torch.randn(oshape, generator=g), _bf(torch.randn(oshape, generator=g))
    P = _bf(dy * torch.where(y.float() > 0, 1.0, SLOPE))
    xad, xbd = xa.to(DEV), (None if xb is None else xb.to(DEV))
    dw, db = ops.conv3d_bwd_weight_bf16(xad, xbd, P.to(DEV), geom)
    rw, rb = oracle.conv3d_bwd_weight(xa.double(), None if xb is None else xb.double(), P.double(), N, Di, Hi, Wi, Ca,
                                      Cb, Cout, stride=s, ups=ups)
    assert_grad(dw.cpu().numpy(), rw, "dw")
    assert_grad(db.cpu().numpy(), rb, "db")
    dw2, db2 = ops.conv3d_bwd_weight(xad, xbd, dy.to(DEV), y.to(DEV), geom, slope=SLOPE)
    assert torch.equal(dw2, dw) and torch.equal(db2, db)


# Forward and input gradient: one short of, equal to and one past a tile of
# 16 x 8 WR voxels and a z chunk; every channel pattern (up to 8, 16, 32 and
# more channels, multiples of 4 that are not of 8), part a upsampled or not,
# one to five output-channel tiles, both strides.
DATA_CASES = [
    (1, 1, 1, 1, 4, 0, 4, 1, False),
    (1, 3, 31, 17, 8, 0, 16, 1, False),
    (2, 2, 33, 16, 12, 0, 20, 1, False),
    (1, 7, 9, 15, 16, 0, 48, 1, False),
    (1, 5, 8, 33, 4, 0, 52, 1, False),
    (1, 4, 34, 18, 32, 16, 12, 1, True),
    (1, 2, 30, 32, 16, 8, 16, 1, True),
    (1, 2, 18, 34, 28, 4, 16, 1, True),
    (1, 4, 16, 14, 64, 32, 28, 1, True),
    (1, 3, 17, 15, 32, 0, 16, 1, False),
    (1, 3, 15, 17, 36, 20, 24, 1, False),
    (1, 2, 9, 5, 40, 24, 96, 1, False),
    (1, 2, 17, 16, 32, 32, 80, 1, False),
    (1, 3, 8, 16, 68, 0, 64, 1, False),
    (2, 20, 40, 34, 16, 8, 64, 1, True),  # wide layers: z chunks of 2 slices, then of 3
    (2, 40, 40, 34, 16, 8, 64, 1, True),
    (1, 9, 15, 33, 16, 0, 32, 2, False),
    (1, 4, 17, 31, 8, 0, 64, 2, False),
    (2, 3, 16, 35, 32, 0, 48, 2, False),
    (1, 5, 9, 17, 64, 32, 20, 2, False),
    (1, 4, 5, 7, 36, 0, 64, 2, False),
    (1, 6, 18, 34, 32, 16, 40, 2, True),
    (1, 4, 10, 6, 24, 0, 12, 2, True),
]


@pytest.mark.parametrize("case", DATA_CASES)
def test_forward_and_input_gradient(case):
    print(f"[conv fwd/dgrad tiles {case}]", flush=True)
    N, Di, Hi, Wi, Ca, Cb, Cout, s, ups = case
    xa, xb, w, b, geom = _case(*case, seed=7)
    wbf, wt = ops.conv3d_weight_prep(w.to(DEV))
    wq = wbf.cpu().double()
    xad, xbd = xa.to(DEV), (None if xb is None else xb.to(DEV))
    ybf, yf = ops.conv3d_fwd(xad, xbd, wbf, b.to(DEV), geom, act=True, slope=SLOPE, want_f32=True)
    ref = oracle.conv3d_fwd(xa.double(), None if xb is None else xb.double(), wq, b.double(), N, Di, Hi, Wi, Ca, Cb,
                            Cout, stride=s, ups=ups, act=True, slope=SLOPE)
    assert_grad(yf.cpu().numpy(), ref, "fwd")
    assert torch.equal(ybf.cpu(), _bf(yf.cpu()))
    dy = torch.randn(yf.shape, generator=torch.Generator().manual_seed(8))
    P = ops.conv3d_act_grad(dy.to(DEV), ybf, slope=SLOPE)
    dx = ops.conv3d_bwd_data_bf16(P, wt, geom)
    rdx = oracle.conv3d_bwd_data(P.cpu().double(), wq, N, Di, Hi, Wi, Ca, Cb, Cout, stride=s)
    assert_grad(dx.cpu().numpy(), rdx, "dx")
    acc = ops.conv3d_bwd_data(dy.to(DEV), ybf, wt, geom, slope=SLOPE, dx=dx.clone(), accumulate=True)
    assert torch.equal(acc, dx + dx)


@pytest.mark.parametrize("Ca,Cb,Cout,s,ups", [(4, 0, 16, 1, False), (16, 0, 16, 1, False), (32, 16, 16, 1, True),
                                              (32, 32, 64, 1, False), (16, 0, 32, 2, False), (64, 0, 32, 2, False)])
def test_infinite_input_stays_in_its_window(Ca, Cb, Cout, s, ups):
    """An infinite activation reaches the outputs whose 3^3 window holds it, as +-inf, and no other."""
    print(f"[conv inf {Ca} {Cb} {Cout} {s} {ups}]", flush=True)
    n = (6, 18, 20)
    xa, xb, w, b, geom = _case(1, *n, Ca, Cb, Cout, s, ups, seed=9)
    w = w.abs() + 0.01
    (xa if xb is None else xb)[0, 2, 9, 10, 3] = float("inf")
    y = ops.conv3d_fwd(xa.to(DEV), None if xb is None else xb.to(DEV), _bf(w).to(DEV), b.to(DEV), geom,
                       want_bf16=False, want_f32=True)[0].cpu()
    hit = torch.zeros(y.shape, dtype=torch.bool)
    z, yy, x = (slice(-(-(c - 1) // s), (c + 1) // s + 1) for c in (2, 9, 10))
    hit[z, yy, x] = True
    assert torch.equal(torch.isinf(y), hit) and not torch.isnan(y).any()
