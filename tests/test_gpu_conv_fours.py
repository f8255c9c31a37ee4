"""GPU parity of the convolutions with channels in fours, of thin upsampled
inputs, and of the tile shapes of three output-channel tiles: one short of, equal
to and one past a tile, both strides.  Operands, oracle and tolerance as in
test_gpu_conv_tiles.py."""
import pytest
import torch

import oracle
from paper_2509_25044_amd import ops
from parity_util import assert_grad
from test_gpu_conv import DEV, SLOPE, _bf, _case

pytestmark = pytest.mark.gpu

# N, Di, Hi, Wi, Ca, Cb, Cout, stride, ups
CASES = [
    (1, 2, 2, 2, 4, 0, 4, 1, True),      # upsampled, up to 8 channels
    (1, 4, 18, 34, 4, 0, 16, 1, True),
    (2, 6, 14, 30, 8, 0, 36, 1, True),
    (1, 4, 16, 32, 8, 0, 48, 1, True),
    (1, 6, 18, 34, 4, 0, 16, 2, True),
    (1, 4, 34, 66, 8, 0, 52, 2, True),
    (1, 4, 18, 34, 12, 0, 20, 1, True),  # ... up to 16
    (1, 2, 16, 32, 16, 0, 4, 1, True),
    (2, 6, 10, 18, 16, 0, 64, 1, True),
    (1, 6, 18, 30, 12, 0, 28, 2, True),
    (1, 4, 34, 66, 16, 0, 16, 2, True),
    (1, 3, 17, 33, 20, 4, 16, 1, False),  # fours: one, two, three and four tiles of output channels
    (1, 4, 16, 32, 20, 4, 16, 1, True),
    (1, 3, 7, 15, 36, 0, 32, 1, False),
    (1, 4, 10, 18, 28, 12, 44, 1, True),
    (1, 2, 9, 17, 68, 0, 68, 1, False),
    (1, 5, 15, 33, 20, 4, 16, 2, False),
    (1, 4, 18, 34, 20, 4, 16, 2, True),
    (1, 5, 33, 35, 68, 0, 64, 2, False),
    (1, 4, 34, 30, 60, 4, 40, 2, True),
]


@pytest.mark.parametrize("case", CASES)
def test_forward_and_input_gradient(case):
    print(f"[conv fours {case}]", flush=True)
    N, Di, Hi, Wi, Ca, Cb, Cout, s, ups = case
    xa, xb, w, b, geom = _case(*case, seed=17)
    wbf, wt = ops.conv3d_weight_prep(w.to(DEV))
    wq = wbf.cpu().double()
    xad, xbd = xa.to(DEV), (None if xb is None else xb.to(DEV))
    ybf, yf = ops.conv3d_fwd(xad, xbd, wbf, b.to(DEV), geom, act=True, slope=SLOPE, want_f32=True)
    ref = oracle.conv3d_fwd(xa.double(), None if xb is None else xb.double(), wq, b.double(), N, Di, Hi, Wi, Ca, Cb,
                            Cout, stride=s, ups=ups, act=True, slope=SLOPE)
    assert_grad(yf.cpu().numpy(), ref, "fwd")
    assert torch.equal(ybf.cpu(), _bf(yf.cpu()))
    dy = torch.randn(yf.shape, generator=torch.Generator().manual_seed(18))
    P = ops.conv3d_act_grad(dy.to(DEV), ybf, slope=SLOPE)
    dx = ops.conv3d_bwd_data_bf16(P, wt, geom)
    rdx = oracle.conv3d_bwd_data(P.cpu().double(), wq, N, Di, Hi, Wi, Ca, Cb, Cout, stride=s)
    assert_grad(dx.cpu().numpy(), rdx, "dx")
    assert torch.equal(ops.conv3d_bwd_data(dy.to(DEV), ybf, wt, geom, slope=SLOPE), dx)


@pytest.mark.parametrize("Ca,Cb,Cout,s,ups", [(4, 0, 16, 1, True), (16, 0, 16, 1, True), (8, 0, 32, 2, True),
                                              (20, 4, 16, 1, False), (20, 4, 16, 1, True), (20, 4, 32, 2, False)])
def test_infinite_input_stays_in_its_window(Ca, Cb, Cout, s, ups):
    """An infinite activation reaches the outputs whose 3^3 window holds it, as +-inf, and no other."""
    print(f"[conv fours inf {Ca} {Cb} {Cout} {s} {ups}]", flush=True)
    xa, xb, w, b, geom = _case(1, 6, 18, 20, Ca, Cb, Cout, s, ups, seed=19)
    at = (1, 4, 5) if ups else (2, 9, 10)
    xa[0, at[0], at[1], at[2], 3] = float("inf")
    y = ops.conv3d_fwd(xa.to(DEV), None if xb is None else xb.to(DEV), _bf(w.abs() + 0.01).to(DEV), b.to(DEV), geom,
                       want_bf16=False, want_f32=True)[0].cpu()
    hit = torch.zeros(y.shape, dtype=torch.bool)
    lo, hi = [2 * c if ups else c for c in at], [2 * c + 1 if ups else c for c in at]
    z, yy, x = (slice(-(-(a - 1) // s), (c + 1) // s + 1) for a, c in zip(lo, hi))
    hit[z, yy, x] = True
    assert torch.equal(torch.isinf(y), hit) and not torch.isnan(y).any()


def test_three_tiles_on_either_side_of_a_million_voxels():
    """Waves of 4 rows up to 2^20 output voxels, of 8 beyond: the same sums, so the same bits."""
    print("[conv three tiles]", flush=True)
    shape = (60, 98, 100)
    g = torch.Generator(device=DEV).manual_seed(20)
    x = torch.randn((2,) + shape + (16,), generator=g, device=DEV).bfloat16()
    w, wt = ops.conv3d_weight_prep(torch.randn((48, 27, 16), generator=g, device=DEV) * 0.05)
    b = torch.randn(48, generator=g, device=DEV)
    one, two = ops.conv_geom(1, *shape, 16, 0, 48, 1, False), ops.conv_geom(2, *shape, 16, 0, 48, 1, False)
    y = ops.conv3d_fwd(x, None, w, b, two, want_bf16=False, want_f32=True)
    back1, back2 = ops.conv_geom(1, *shape, 48, 0, 16, 1, False), ops.conv_geom(2, *shape, 48, 0, 16, 1, False)
    _, wt48 = ops.conv3d_weight_prep(torch.randn((16, 27, 48), generator=g, device=DEV) * 0.05)
    dx = ops.conv3d_bwd_data_bf16(x, wt48, back2)
    for n in range(2):
        xn = x[n:n + 1].contiguous()
        assert torch.equal(ops.conv3d_fwd(xn, None, w, b, one, want_bf16=False, want_f32=True)[0], y[n])
        assert torch.equal(ops.conv3d_bwd_data_bf16(xn, wt48, back1)[0], dx[n])
