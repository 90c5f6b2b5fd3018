"""The library's dispatch rules, asked on the CPU: which kernel takes a call,
and with what split, so that a rule that moves shows here."""
import ctypes
from ctypes import c_int, c_int64

import numpy as np
import pytest

import paper_2605_22850_amd as oc
from tests.attention_cases import BATCHES, BY_PLAN, RAGGED


def gemm_rows(M, K, N, has_workspace):
    """Number of ranges the few-row kernels split K into; 0: the GEMM library."""
    f = oc.lib().oc_internal_gemm_rows
    f.argtypes = [c_int64, c_int64, c_int64, c_int, ctypes.POINTER(c_int64)]
    n = c_int64()
    f(M, K, N, has_workspace, ctypes.byref(n))
    return n.value


def test_no_product_is_split_without_a_workspace():
    """Calls on the per-thread stream, and those past the number of workspaces,
    have none: their products are unsplit or the library's."""
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


def attention_plan(nq, nkv, d, Tp, Ts):
    """(tile rows, row tiles, key blocks, splits, blocks per split)"""
    lay = oc.Layout(1, nq, nkv, d, 16, 16, max(1, -(-Tp // 16))).c()
    out = (c_int64 * 5)()
    assert oc.lib().oc_internal_attention_plan(ctypes.byref(lay), c_int64(Tp), c_int64(Ts), out) == 0
    return tuple(out)


def place_of_partial_page(Tp, n_blocks, per_range, pages_per_block):
    """Where in its range of key blocks the prefix's partial page lies."""
    block = Tp // 16 // pages_per_block
    at, last = block % per_range, min(per_range, n_blocks - block // per_range * per_range) - 1
    return "only" if last == 0 else "first" if at == 0 else "last" if at == last else "middle"


@pytest.mark.parametrize("tile,d,split", list(BY_PLAN))
def test_attention_cases_take_the_kernel_they_name(tile, d, split):
    odd = set()
    for case in BY_PLAN[tile, d, split]:
        rows, _, _, n_split, _ = attention_plan(*case)
        assert (rows, case[2], n_split > 1) == (tile, d, split), (case, rows, n_split)
        odd.add(case[1] * n_split % 8 != 0)
    assert True in odd or (tile, d, split) == (256, 64, False)      # groups that do not load the XCDs evenly


@pytest.mark.parametrize("tile,d", list(RAGGED))
def test_ragged_prefixes_take_the_kernel_they_name(tile, d):
    places = set()
    for case in RAGGED[tile, d]:
        rows, _, n_blocks, _, per_range = attention_plan(*case)
        assert (rows, case[2]) == (tile, d), (case, rows)
        assert tile < 256 or per_range >= 5
        places.add(place_of_partial_page(case[3], n_blocks, per_range, 4 if tile == 256 else 2))
    assert {case[3] % 16 for case in RAGGED[tile, d]} == {1, 5, 8, 15}
    assert tile < 256 or places == {"first", "middle", "last"}


def test_batches_cover_ranges_of_one_to_many_blocks():
    places, slots = set(), set()
    for nq, nkv, Tp, Ts, per_range in BATCHES:
        for d in (64, 128):
            n = len(Tp)
            lay = oc.Layout(1, nq, nkv, d, 16, 16, 1000).c()
            out = (c_int64 * (5 * n))()
            assert oc.lib().oc_internal_attention_batch_plan(ctypes.byref(lay), n, (c_int64 * n)(*Tp), (c_int64 * n)(*Ts),
                                                             out) == 0
            plans = [out[5 * i:5 * i + 5] for i in range(n)]
            assert {p[0] for p in plans} == {256} and {p[4] for p in plans} == per_range, (nq, nkv, plans)
            for t, p in zip(Tp, plans):
                if t % 16:
                    places.add(place_of_partial_page(t, p[2], p[4], 4))
                    slots.add(t % 16)
    assert places == {"only", "first", "middle", "last"} and slots >= {1, 5, 8, 15}
