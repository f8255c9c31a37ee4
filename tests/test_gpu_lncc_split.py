"""GPU parity of the two-kernel LNCC adjoint (windows 7 and 9) and of its border
with the one-kernel form: widths either side of its row runs (4), thread counts
(64, 128, 256) and limit (512), heights either side of its chunks of 8 and 16
rows, an ROI, no displacement, and an infinite voxel."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25044_amd import ops, synth
from parity_util import assert_grad, assert_loss

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _pair(shape, seed=3):
    p = synth.make_pair(synth.PairSpec(shape, (3.0, 6.0), 2.0, texture_std=0.05), seed=seed)
    return p["F"], p["M"], (-0.7 * p["d"]).contiguous()


CASES = [((40, 17, 63), 7, None), ((41, 16, 65), 9, None), ((40, 33, 127), 9, None), ((40, 15, 130), 7, None),
         ((60, 31, 255), 9, None), ((60, 9, 258), 7, None), ((64, 8, 512), 9, None), ((64, 24, 513), 7, None),
         ((48, 40, 44), 7, ((5, 40), (3, 37), (8, 44))), ((50, 48, 56), 9, ((0, 50), (10, 11), (0, 56)))]


@pytest.mark.parametrize("shape,window,roi", CASES)
def test_matches_oracle(shape, window, roi):
    print(f"[lncc split {shape} w={window} roi={roi}]", flush=True)
    F, M, u = _pair(shape)
    r6 = None if roi is None else [v for k in roi for v in k]
    for disp in (u, None):
        g, l = ops.warp_lncc_bwd(F.to(DEV), M.to(DEV), None if disp is None else disp.to(DEV), window=window, roi=roi)
        lr, gr = oracle.lncc(F.numpy(), M.numpy(), None if disp is None else disp.numpy(), roi=r6, window=window)
        assert_loss(float(l.item()), lr, "loss")
        assert_grad(g.cpu().numpy(), gr, "grad")
    # no loss asked for: the same gradient; a scale on the device: linear
    g2, l2 = ops.warp_lncc_bwd(F.to(DEV), M.to(DEV), None, window=window, roi=roi, want_loss=False)
    assert l2 is None and torch.equal(g2, g)
    g3, _ = ops.warp_lncc_bwd(F.to(DEV), M.to(DEV), None, window=window, roi=roi, grad_scale=torch.full((1,), 2.0, device=DEV))
    assert torch.equal(g3, 2 * g)


def test_infinite_voxel_reaches_its_windows_only():
    shape, window = (48, 48, 56), 7
    F, M, u = _pair(shape)
    u.zero_()
    F[20, 22, 24] = float("inf")
    g, _ = ops.warp_lncc_bwd(F.to(DEV), M.to(DEV), u.to(DEV), window=window)
    far = torch.ones(shape, dtype=torch.bool)
    far[20 - 6:20 + 7, 22 - 6:22 + 7, 24 - 6:24 + 7] = False
    assert torch.isfinite(g.cpu()[:, far]).all()
    F[20, 22, 24] = 0.5
    g0, _ = ops.warp_lncc_bwd(F.to(DEV), M.to(DEV), u.to(DEV), window=window)
    assert_grad(g.cpu()[:, far].numpy(), g0.cpu()[:, far].numpy().astype(np.float64), "beyond the windows")
