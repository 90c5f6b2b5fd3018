"""The library's dispatch rules, asked on the CPU: which kernel takes a call,
and with what split, so that a rule that moves shows here."""
import ctypes
from ctypes import c_int, c_int64

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
