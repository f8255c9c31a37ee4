"""GPU: bf16 operands at addresses that are multiples of 8 but not of 16 bytes,
which the convolutions' entry points take, give the bits that 16-byte aligned
copies give: every output is the same sum in the same order whichever width its
operands are loaded in."""
import pytest
import torch

from paper_2509_25044_amd import ops
from test_gpu_conv import DEV, SLOPE, _bf, _case

pytestmark = pytest.mark.gpu


def _at8(t):
    """A copy of t that begins 8 bytes into a 16-byte aligned allocation."""
    if t is None:
        return None
    buf = torch.empty(t.numel() + 4, dtype=t.dtype, device=t.device)
    assert buf.data_ptr() % 16 == 0
    v = buf[4:].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == 8
    return v


# wide stride-1 layers (one to six output tiles, part a upsampled or not, chunks
# of 1 to 3 slices), the tile kernel's patterns, stride 2
CASES = [
    (1, 5, 18, 34, 32, 16, 64, 1, False),
    (1, 4, 18, 34, 64, 32, 32, 1, True),
    (1, 2, 9, 17, 64, 0, 16, 1, False),
    (2, 40, 40, 34, 16, 8, 64, 1, True),
    (1, 3, 17, 16, 32, 0, 96, 1, False),
    (1, 6, 18, 34, 32, 16, 16, 1, True),
    (1, 4, 9, 33, 16, 0, 16, 1, False),
    (1, 3, 9, 17, 8, 0, 4, 1, False),
    (1, 5, 17, 33, 16, 0, 32, 2, False),
    (1, 6, 10, 18, 64, 32, 128, 2, True),
]


@pytest.mark.parametrize("case", CASES)
def test_operands_at_8_bytes(case):
    print(f"[conv 8-byte operands {case}]", flush=True)
    N, Di, Hi, Wi, Ca, Cb, Cout, s, ups = case
    xa, xb, w, b, geom = _case(*case, seed=21)
    xa, xb, b = xa.to(DEV), (None if xb is None else xb.to(DEV)), b.to(DEV)
    wbf, wt = ops.conv3d_weight_prep(w.to(DEV))
    y = ops.conv3d_fwd(xa, xb, wbf, b, geom, act=True, slope=SLOPE)
    dy = torch.randn(y.shape, generator=torch.Generator().manual_seed(22)).to(DEV)
    P = ops.conv3d_act_grad(dy, y, slope=SLOPE)
    dx = ops.conv3d_bwd_data_bf16(P, wt, geom)
    dw, db = ops.conv3d_bwd_weight_bf16(xa, xb, P, geom)
    for xa2, xb2, w2 in ((_at8(xa), _at8(xb), _at8(wbf)), (_at8(xa), xb, wbf), (xa, _at8(xb), wbf), (xa, xb, _at8(wbf))):
        y2 = torch.empty(y.numel() + 4, dtype=y.dtype, device=DEV)[4:].view(y.shape)
        ops.conv3d_fwd(xa2, xb2, w2, b, geom, act=True, slope=SLOPE, y_bf16=y2)
        assert torch.equal(y2, y)
    assert torch.equal(ops.conv3d_bwd_data_bf16(P, _at8(wt), geom), dx)
    assert torch.equal(ops.conv3d_bwd_data(dy, _at8(y), _at8(wt), geom, slope=SLOPE), dx)
    dw2, db2 = ops.conv3d_bwd_weight_bf16(_at8(xa), _at8(xb), _at8(P), geom)
    assert torch.equal(dw2, dw) and torch.equal(db2, db)
    dw3, db3 = ops.conv3d_bwd_weight(_at8(xa), _at8(xb), dy, _at8(y), geom, slope=SLOPE)
    assert torch.equal(dw3, dw) and torch.equal(db3, db)
