"""GPU parity where a launch plan cuts a small volume into z chunks of a slice
or two: every chunk's halo, the last short chunk, and volumes
one slice either side of a change of the chunk length."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25044_amd import ops, synth
from parity_util import assert_grad, assert_loss

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _pair(shape, seed):
    p = synth.make_pair(synth.PairSpec(shape, (3.0, 6.0), 2.0), seed=seed)
    return p["F"], p["M"], (-0.7 * p["d"]).contiguous()


@pytest.mark.parametrize("shape,window", [((2, 25, 33), 3), ((13, 24, 32), 9), ((37, 17, 65), 5),
                                          ((40, 48, 56), 7), ((3, 25, 33), 15), ((61, 70, 90), 11),
                                          ((33, 130, 257), 13)])
def test_lncc_short_chunks(shape, window):
    print(f"[lncc short chunks {shape} w={window}]", flush=True)
    F, M, u = _pair(shape, 5)
    g, l = ops.warp_lncc_bwd(F.to(DEV), M.to(DEV), u.to(DEV), window=window)
    lr, gr = oracle.lncc(F.numpy(), M.numpy(), u.numpy(), window=window)
    assert_loss(float(l.item()), lr, "loss")
    assert_grad(g.cpu().numpy(), gr, "grad")
    lf = ops.warp_lncc_fwd(F.to(DEV), M.to(DEV), u.to(DEV), window=window)
    assert_loss(float(lf.item()), lr, "forward")


@pytest.mark.parametrize("shape,bins", [((3, 5, 70), 32), ((5, 9, 64), 100), ((21, 30, 40), 8), ((35, 66, 130), 64)])
def test_mi_short_chunks(shape, bins):
    print(f"[mi short chunks {shape} bins={bins}]", flush=True)
    F, M, u = _pair(shape, 6)
    l, st = ops.warp_mi_fwd(F.to(DEV), M.to(DEV), u.to(DEV), bins=bins)
    g = ops.warp_mi_bwd(F.to(DEV), M.to(DEV), u.to(DEV), st, bins=bins)
    lr, _, gr = oracle.mi(F.numpy(), M.numpy(), u.numpy(), bins=bins)
    assert_loss(float(l.item()), lr, "loss")
    assert_grad(g.cpu().numpy(), gr, "grad")


@pytest.mark.parametrize("shape", [(1, 7, 9), (2, 16, 64), (17, 33, 65), (40, 48, 56)])
@pytest.mark.parametrize("sigma", [0.3, 1.0, 2.0])
def test_smoothing_short_chunks(shape, sigma):
    print(f"[smooth short chunks {shape} sigma={sigma}]", flush=True)
    x = torch.randn((3,) + shape, generator=torch.Generator().manual_seed(7))
    out = ops.gaussian_smooth(x.to(DEV), sigma).cpu().numpy().astype(np.float64)
    ref = oracle.gaussian_smooth(x.numpy(), sigma)
    assert np.abs(out - ref).max() <= 1e-6 * max(1.0, np.abs(ref).max())


# LDS histograms: the widest of 256-thread blocks and the first of 1024, one
# copy at the edge of two blocks per CU, the largest whole histogram and the
# first cut into two groups of F bins, three and four groups, both estimators
@pytest.mark.parametrize("bins", [56, 57, 68, 69, 98, 99, 128, 129, 140, 141, 142, 199, 200, 213, 256])
@pytest.mark.parametrize("shape,roi", [((9, 21, 70), None), ((18, 40, 34), ((2, 17), (3, 35), (1, 33)))])
def test_mi_histogram_sizes(bins, shape, roi):
    print(f"[mi histogram {shape} bins={bins} roi={roi}]", flush=True)
    F, M, u = _pair(shape, 8)
    r6 = None if roi is None else [v for k in roi for v in k]
    l, st = ops.warp_mi_fwd(F.to(DEV), M.to(DEV), u.to(DEV), bins=bins, roi=roi)
    g = ops.warp_mi_bwd(F.to(DEV), M.to(DEV), u.to(DEV), st, bins=bins, roi=roi)
    lr, _, gr = oracle.mi(F.numpy(), M.numpy(), u.numpy(), bins=bins, roi=r6)
    assert_loss(float(l.item()), lr, "loss")
    assert_grad(g.cpu().numpy(), gr, "grad")
    l2, st2 = ops.warp_mi_fwd(F.to(DEV), M.to(DEV), u.to(DEV), bins=bins, roi=roi)
    assert torch.equal(st, st2) and torch.equal(l, l2)  # integer sums: the same bits every time
    pmf = st[bins * bins:2 * bins * bins].double().cpu()
    assert abs(float(pmf.sum()) - 1.0) < 1e-5
