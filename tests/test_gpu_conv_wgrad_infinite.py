"""GPU: an infinite activation in the last row and column of a layer's input
reaches the weight gradient's taps that pair it with an output, and no other: not
the taps that would need an output past the last one, nor other channels."""
import pytest
import torch

from paper_2509_25044_amd import ops
from test_gpu_conv import DEV, SLOPE, _case

pytestmark = pytest.mark.gpu


def _reached(i, n_out, stride):
    """Taps d of one axis with an output o at stride o + d - 1 = i, for any of the input indices i."""
    return [any((v + 1 - d) % stride == 0 and 0 <= (v + 1 - d) // stride < n_out for v in i) for d in range(3)]


# outputs one short of, equal to and one past a tile's 32 columns and 8 or 4 rows
@pytest.mark.parametrize("case", [(1, 4, 7, 31, 16, 0, 16, 1, False), (1, 3, 8, 32, 16, 0, 96, 1, False),
                                  (2, 4, 9, 33, 8, 4, 48, 1, False), (1, 6, 10, 18, 32, 16, 16, 1, True),
                                  (1, 6, 10, 34, 16, 0, 32, 2, False), (1, 5, 8, 64, 32, 0, 64, 2, False),
                                  (1, 5, 9, 65, 16, 8, 32, 2, False), (2, 6, 6, 66, 32, 16, 16, 2, True)])
@pytest.mark.parametrize("part", ["a", "b"])
def test_last_row_and_column(case, part):
    print(f"[conv wgrad inf {case} {part}]", flush=True)
    N, Di, Hi, Wi, Ca, Cb, Cout, s, ups = case
    if part == "b" and not Cb:
        pytest.skip("no part b")
    xa, xb, _, _, geom = _case(*case, seed=31)
    out = ops.conv_out_shape(geom)
    P = torch.randn((N,) + out + (Cout,), generator=torch.Generator().manual_seed(32)).bfloat16().to(DEV)
    x = xa if part == "a" else xb
    c = 3 if part == "a" else Ca + 3
    f = 2 if ups and part == "a" else 1  # fine voxels of one stored voxel, per axis
    z = x.shape[1] // 2

    def gradients(v):
        x[N - 1, z, -1, -1, 3] = v
        a, b = xa.to(DEV), None if xb is None else xb.to(DEV)
        return ops.conv3d_bwd_weight_bf16(a, b, P, geom)

    dw0, db0 = gradients(0.0)
    dw, db = gradients(float("inf"))
    hit = torch.zeros(Cout, 27, Ca + Cb, dtype=torch.bool)
    tz = _reached([f * z + k for k in range(f)], out[0], s)
    ty = _reached([Hi - 1 - k for k in range(f)], out[1], s)
    tx = _reached([Wi - 1 - k for k in range(f)], out[2], s)
    for t in range(27):
        hit[:, t, c] = tz[t // 9] and ty[(t // 3) % 3] and tx[t % 3]
    assert (f == 2 or not all(hit[0, :, c])) and torch.isfinite(dw0).all()  # a stored voxel of 2^3 reaches every tap
    assert torch.equal(torch.isfinite(dw.cpu()), ~hit)
    assert torch.equal(dw.cpu()[~hit], dw0.cpu()[~hit]) and torch.equal(db, db0)
