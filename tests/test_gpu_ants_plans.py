"""GPU parity of the LNCC gradient in the ANTs approximation and of the forward
pass with zero padding where the launch plan cuts small volumes into short z
chunks: chunks of a slice or two, a last chunk that is shorter, several rounds."""
import pytest
import torch

import oracle
from paper_2509_25044_amd import ops, synth
from parity_util import assert_grad, assert_loss

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape,window", [((2, 25, 33), 3), ((13, 24, 32), 9), ((37, 17, 65), 7), ((30, 70, 90), 7),
                                          ((61, 49, 100), 5), ((64, 66, 130), 7)])
@pytest.mark.parametrize("pad", ["border", "zeros"])
def test_short_chunks(shape, window, pad):
    print(f"[ants short chunks {shape} w={window} {pad}]", flush=True)
    p = synth.make_pair(synth.PairSpec(shape, (3.0, 6.0), 2.0, texture_std=0.05), seed=12)
    F, M, u = p["F"], p["M"], (-0.7 * p["d"]).contiguous()
    pm = 1 if pad == "zeros" else 0
    Fd, Md, ud = F.to(DEV), M.to(DEV), u.to(DEV)
    g, l = ops.warp_lncc_bwd(Fd, Md, ud, window=window, pad=pad, ants=True)
    lr, gr = oracle.lncc(F.numpy(), M.numpy(), u.numpy(), window=window, pad=pm, ants=True)
    assert_loss(float(l.item()), lr, "loss")
    assert_grad(g.cpu().numpy(), gr, "grad")
    assert_loss(float(ops.warp_lncc_fwd(Fd, Md, ud, window=window, pad=pad).item()), lr, "forward")
