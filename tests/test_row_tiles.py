"""The row tiles of the transposed sweep: 32-bit sums are no longer than one of 64 tiles."""
import ctypes

import numpy as np
import pytest

import paper_2405_05865_amd as msp


def _tiles(rows, ctiles, fp32):
    f = msp.library()._Z16gemv_t_row_tilesllb
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int64, ctypes.c_bool]
    return f(rows, ctiles, fp32)


@pytest.mark.parametrize("rows", [1, 2, 31, 63, 64, 65, 100, 640, 1024, 2047, 2048, 5000])
@pytest.mark.parametrize("ctiles", [1, 3, 32, 33, 2048, 5000])
def test_tiles_fill_the_chip_within_the_partials(rows, ctiles):
    fill = -(-2048 // ctiles)
    for fp32, most in ((True, min(64, rows)), (False, min(64, rows // 32))):
        assert _tiles(rows, ctiles, fp32) == max(1, min(fill, most))


@pytest.mark.parametrize("rows", [100, 300, 640, 1024])
def test_fp32_sums_keep_their_length(rows):
    # the product as the kernel forms it: FP32 multiply-adds within a tile, FP64 over the tiles
    g = np.random.default_rng(rows)
    a = g.standard_normal((rows, 2000)).astype(np.float32)
    x = g.standard_normal(rows).astype(np.float32)

    def product(tiles):
        per = -(-rows // tiles)
        out = np.zeros(a.shape[1])
        for r0 in range(0, rows, per):
            acc = np.zeros(a.shape[1], np.float32)
            for r in range(r0, min(rows, r0 + per)):
                acc = (acc + a[r].astype(np.float64) * np.float64(x[r])).astype(np.float32)
            out += acc
        return out

    want = a.T.astype(np.float64) @ x.astype(np.float64)
    err = [np.linalg.norm(product(t) - want) for t in (_tiles(rows, 2, True), min(64, rows))]
    assert err[0] <= err[1]
