"""CPU: which grids the entry point without a workspace takes does not depend on
how finely a plan cuts a small volume.  A wide window (w >= 11) needs 8 doubles
per voxel and one per block; with z chunks of at least 32 slices, as many blocks
as fit the rest of the array, every grid below fits it."""
import ctypes as C

import pytest

from paper_2509_25044_amd import _lib, ops

LIMIT = 65536  # doubles; two more hold the checked-mode flag


def _need(shape, window):
    L = _lib.lib()
    g, p = ops.make_grid(shape, None), ops.lncc_params(window)
    return L.ffdp_lncc_workspace_bytes(C.byref(g), C.byref(p)) // 8 - 2


@pytest.mark.parametrize("shape", [(102, 80, 1), (204, 5, 8), (34, 48, 5), (13, 9, 70), (227, 6, 6), (2, 89, 46),
                                   (113, 72, 1), (36, 113, 2), (272, 10, 3), (372, 11, 2)])
@pytest.mark.parametrize("window", [11, 13, 15])
def test_wide_windows_at_the_limit(shape, window):
    D, H, W = shape
    columns = -(-H // 4) * -(-W // 64)
    assert 8 * D * H * W + columns * max(1, D // 32) <= LIMIT
    assert _need(shape, window) <= LIMIT


def test_every_grid_that_32_slice_chunks_fit():
    for D in range(1, 420, 7):
        for H in (1, 3, 4, 5, 9, 16, 40, 90):
            W = (LIMIT // (8 * D * H))
            for w in (W, W - 1):
                if w < 1:
                    continue
                columns = -(-H // 4) * -(-w // 64)
                if 8 * D * H * w + columns * max(1, D // 32) <= LIMIT:
                    assert _need((D, H, w), 11) <= LIMIT, (D, H, w)
