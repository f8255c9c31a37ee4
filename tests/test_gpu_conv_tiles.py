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
