"""The library's dispatch rules, asked on the CPU: which kernel takes a call,
and with what split, so that a rule that moves shows here."""
import ctypes
from ctypes import c_int, c_int64

import numpy as np
import pytest

import paper_2605_22850_amd as oc


def gemm_rows(M, K, N, has_workspace):
    """Number of ranges the few-row kernels split K into; 0: the GEMM library."""
    f = oc.lib().oc_internal_gemm_rows
    f.argtypes = [c_int64, c_int64, c_int64, c_int, ctypes.POINTER(c_int64)]
    n = c_int64()
    f(M, K, N, has_workspace, ctypes.byref(n))
    return n.value


def test_no_product_is_split_without_a_workspace():
    """Captured calls and the per-thread stream have no workspace of their own:
    their products are unsplit or the library's."""
    split = unsplit = 0
    for M in (1, 31, 32, 33, 64, 65, 128, 129, 256, 257, 512, 513, 4096):
        for K in (64, 192, 256, 512, 1792, 4096, 14336, 28672):
            for N in (128, 384, 512, 1024, 4096, 6144, 28672):
                with_ws, without = gemm_rows(M, K, N, 1), gemm_rows(M, K, N, 0)
                assert without in (0, 1), (M, K, N)
                # unsplit products keep their kernel
                assert without == (with_ws if with_ws <= 1 else 0), (M, K, N)
                split += with_ws > 1
                unsplit += without == 1
    assert split > 50 and unsplit > 20


def test_few_row_products_fit_the_cus_at_once():
    """Column tiles of 128 in one round over 256 CUs up to 64 rows, over half of
    them to 512 rows (tiles of 128 rows at 257-384, else of 256)."""
    for M, K, N, ours in ((1, 8192, 57344, False), (64, 3584, 37888, False), (64, 4096, 32768, True),
                          (64, 4096, 32896, False), (64, 4096, 28672, True), (65, 4096, 28672, False),
                          (128, 4096, 16384, True), (129, 4096, 16512, False), (256, 4096, 6144, True),
                          (384, 4096, 6144, False), (385, 4096, 6144, True), (512, 14336, 4096, True),
                          (513, 14336, 4096, False), (32, 4096, 100, False), (32, 100, 4096, False)):
        assert (gemm_rows(M, K, N, 1) > 0) == ours, (M, K, N)


def tile_order(tile_rows, m_tiles, groups):
    """(group, row tile) of each workgroup of an attention launch, in order."""
    f = oc.lib().oc_internal_attention_tiles
    f.restype = c_int64
    out = np.empty((2 * (groups + 8) * (m_tiles + 8), 2), np.int32)
    n = f(tile_rows, m_tiles, groups, 1, out.ctypes.data_as(ctypes.c_void_p), c_int64(out.shape[0]))
    assert n <= out.shape[0] and n % 8 == 0
    return out[:n]


@pytest.mark.parametrize("tile_rows", [32, 64, 256])
def test_every_row_tile_has_one_workgroup(tile_rows):
    for groups in [*range(1, 34), 47, 60, 63, 64, 108, 122, 128, 129]:
        for m_tiles in (1, 2, 3, 4, 5, 7, 8, 16, 31, 32, 33, 64):
            order = tile_order(tile_rows, m_tiles, groups)
            real = order[order[:, 0] >= 0]
            assert sorted(map(tuple, real)) == [(g, m) for g in range(groups) for m in range(m_tiles)], \
                (groups, m_tiles)
            for g in {0, groups - 1}:           # a group's last row tile comes first
                assert list(real[real[:, 0] == g, 1]) == list(range(m_tiles - 1, -1, -1))


def test_groups_that_stay_on_one_xcd():
    """By XCD: a multiple of 8 groups; for the small tiles also more than 8
    groups whose busiest XCD runs all its workgroups at once or that load the
    XCDs within 1/15 of evenly."""
    def by_xcd(tile_rows, m_tiles, groups):
        order = tile_order(tile_rows, m_tiles, groups)
        return all(len(set(np.flatnonzero(order[:, 0] == g) % 8)) == 1 for g in range(groups))
    for rows, mt, groups, want in ((256, 16, 8, True), (256, 4, 60, False), (256, 2, 12, False), (32, 4, 60, True),
                                   (64, 4, 60, True), (32, 5, 60, True), (32, 16, 15, True), (64, 17, 15, True),
                                   (64, 17, 14, False), (32, 8, 28, True), (32, 9, 28, False), (64, 5, 90, True),
                                   (32, 4, 6, False), (32, 16, 9, True), (32, 17, 9, False), (32, 200, 16, True)):
        assert by_xcd(rows, mt, groups) == want, (rows, mt, groups)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tile_rows", [32, 64, 256])
def test_one_ingest_workgroup_fits_beside_the_attention(tile_rows, d):
    """LDS goes out in units of 1280 bytes, 128 to a CU; one ingest workgroup
    shares a CU with an attention workgroup of any tile, two do not."""
    attn, ingest = c_int64(), c_int64()
    oc.lib().oc_internal_lds(tile_rows, d, ctypes.byref(attn), ctypes.byref(ingest))
    held, reserved = -(-attn.value // 1280), -(-ingest.value // 1280)
    assert held + reserved <= 128 < held + 2 * reserved
