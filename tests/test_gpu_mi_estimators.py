"""GPU parity of the larger mutual-information histograms for every estimator,
padding and sampler: 1024-thread blocks (57 bins and more), groups of F bins (141
and more), the approximate estimator's counts at the most bins that LDS holds
(199) and either side, and the composite affine sampler."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25044_amd import ops
from parity_util import assert_grad, assert_loss
from test_gpu_affine import _about_centre, _case, _f32, _rot
from test_gpu_parity import DEV, _mi_case, _rand_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins,hard,pad", [(64, True, "border"), (142, True, "zeros"), (64, False, "zeros"),
                                           (100, False, "zeros"), (142, False, "zeros")])
def test_estimators_and_padding(bins, hard, pad):
    F, M, u = _rand_case((18, 28, 36), 500 + bins)
    _mi_case(F, M, u, bins=bins, hard=hard, pad=pad, roi=((1, 17), (0, 27), (2, 36)), what=f"b{bins}")


@pytest.mark.parametrize("bins", [128, 129, 198, 199, 200, 256])
def test_approximate_counts(bins):
    """Probabilities and loss where the warped image is M itself, so that both sides count the same bins.  (Not the
    gradient: at some bin counts the oracle's weights at a bin's centre are 1e-47 and not 0, and so is its probability
    where no voxel contributes, whose logarithm it uses.)"""
    print(f"[mi approx bins={bins}]", flush=True)
    F, M, _ = _rand_case((18, 28, 36), 500 + bins)
    for roi in (None, ((1, 17), (0, 27), (2, 36))):
        r6 = None if roi is None else [v for k in roi for v in k]
        loss, st = ops.warp_mi_fwd(F.to(DEV), M.to(DEV), None, bins=bins, hard="approx", roi=roi)
        rl, rp, _ = oracle.mi(F.numpy(), M.numpy(), None, roi=r6, bins=bins, hard=2, with_grad=False)
        assert_loss(float(loss.item()), rl, "loss")
        np.testing.assert_allclose(st[bins * bins:2 * bins * bins].cpu().numpy().reshape(bins, bins), rp, rtol=1e-5,
                                   atol=1e-9)


@pytest.mark.parametrize("bins", [64, 65, 100, 142])
def test_composite_sampler(bins):
    print(f"[affine mi bins={bins}]", flush=True)
    shape = (24, 28, 36)
    F, M, u = _case(shape, 33)
    A, t = _about_centre(shape, 1.02 * _rot(0.05, 0.04, -0.06), (0.31, -0.27, 0.45))
    A, t, S = _f32(A), _f32(t), _f32(np.diag([0.9, 1.1, 1.0]))
    Fd, Md, ud = F.to(DEV), M.to(DEV), u.to(DEV)
    loss, st = ops.warp_mi_affine_fwd(Fd, Md, ud, A=A, t=t, S=S, bins=bins)
    gu, gA, gt = ops.warp_mi_affine_bwd(Fd, Md, ud, st, A=A, t=t, S=S, bins=bins, want_grad_u=True)
    rl, rp, rgu, rgA, rgt = oracle.mi_affine(F.numpy(), M.numpy(), u.numpy(), A=A, t=t, S=S, bins=bins, hard=0)
    assert_loss(float(loss.item()), rl, "loss")
    np.testing.assert_allclose(st[bins * bins:2 * bins * bins].cpu().numpy().reshape(bins, bins), rp, rtol=1e-5,
                               atol=1e-9)
    assert_grad(gu.cpu().numpy(), rgu, "grad_u")
    assert np.abs(gA.cpu().numpy() - rgA).max() <= 1e-4 * np.abs(rgA).max()
    assert np.abs(gt.cpu().numpy() - rgt).max() <= 1e-4 * np.abs(rgt).max()
    _, gA2, gt2 = ops.warp_mi_affine_bwd(Fd, Md, ud, st, A=A, t=t, S=S, bins=bins)
    assert torch.equal(gA, gA2) and torch.equal(gt, gt2)
