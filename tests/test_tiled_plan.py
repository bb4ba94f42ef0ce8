"""The rule that picks the tiled kernels' tile shapes and K splits, on 256
compute units (what the library assumes without a device): every shape is
still chosen somewhere, and a choice holds over the sizes around it."""

import ctypes

import pytest
import torch

import paper_2607_16339_amd as lc
from paper_2607_16339_amd import _lib


@pytest.mark.parametrize("size,plan", [
    ((65, 128, 128), (64, 64, 128, 1, True)), ((128, 4096, 12288), (64, 64, 128, 4, True)),
    ((200, 4096, 12288), (128, 64, 128, 2, True)), ((256, 4096, 12288), (128, 64, 128, 2, True)),
    ((333, 4096, 12288), (192, 128, 256, 5, False)), ((512, 4096, 12288), (256, 128, 256, 4, False)),
    ((700, 4096, 12288), (192, 128, 256, 2, False)), ((1024, 4096, 12288), (128, 128, 128, 1, False)),
    ((4096, 4096, 12288), (256, 256, 256, 1, False)), ((8192, 4096, 12288), (256, 256, 256, 1, False)),
    ((400, 3072, 8192), (128, 64, 128, 1, True)), ((333, 3072, 8192), (96, 128, 128, 3, False))])
def test_plan_of_known_sizes(size, plan):
    got = lc.lacache_tiled_plan(*size)
    assert got == plan or torch.cuda.is_available()  # (a device may have other compute units)


def test_plan_stays_within_the_workspace_and_the_kernels():
    """The splits fit the partials that the workspace holds, every split has a
    K-group, the register kernel takes one round and no per-channel scales."""
    for M in (1, 64, 65, 127, 129, 200, 257, 333, 512, 700, 1023, 2000, 5000, 1 << 24):
        for H in (128, 384, 640, 4096, 8192, 16384):
            for I in (128, 384, 2048, 12288, 65536):
                room = lc.lacache_ffn_g_workspace_bytes(M, H, I) - 4 * M * max(H, I) - M * (H + I)
                for scales in (False, True):
                    gu, bm, bn, ks, regs = lc.lacache_tiled_plan(M, H, I, scales)
                    assert gu in (64, 96, 128, 192, 256)
                    assert (bm, bn) in ((256, 256), (128, 256), (128, 128), (64, 128))
                    assert 1 <= ks <= max(1, I // 128) and (ks == 1 or ks * M * H * 4 <= room)
                    assert not regs or ((bm, bn) == (64, 128) and not scales)


def test_plan_arguments():
    p = (ctypes.c_int * 5)()
    L = _lib.lib()
    assert L.lacache_tiled_plan(0, 128, 128, 0, p) == lc.LACACHE_ERR_INVALID_ARG
    assert L.lacache_tiled_plan(64, 128, 128, 0, None) == lc.LACACHE_ERR_INVALID_ARG
    assert L.lacache_tiled_plan(64, 100, 128, 0, p) == lc.LACACHE_ERR_INVALID_ARG
    assert L.lacache_tiled_plan(64, 1 << 20, 128, 0, p) == lc.LACACHE_ERR_UNSUPPORTED
    assert L.lacache_tiled_plan(64, 128, 128, 0, p) == lc.LACACHE_OK


def test_projection_tiles():
    """Streamed up to 128 rows (three slabs to a workgroup where one per CU
    remains), and each of the three tile shapes above."""
    if not torch.cuda.is_available():
        for size, tile in (((32, 12288, 4096), (64, 48)), ((33, 12288, 4096), (64, 16)), ((128, 384, 128), (64, 16)),
                           ((129, 12288, 4096), (128, 128)), ((512, 12288, 4096), (128, 192)),
                           ((1000, 12288, 4096), (256, 192)), ((1280, 12288, 128), (128, 128)),
                           ((1 << 24, 128, 128), (128, 128))):
            assert lc.lacache_linear_tile(*size) == tile, size
    t = (ctypes.c_int * 2)()
    L = _lib.lib()
    assert L.lacache_linear_tile(0, 128, 128, t) == lc.LACACHE_ERR_INVALID_ARG
    assert L.lacache_linear_tile(1, 128, 128, None) == lc.LACACHE_ERR_INVALID_ARG
    assert L.lacache_linear_tile(1, 100, 128, t) == lc.LACACHE_ERR_INVALID_ARG
