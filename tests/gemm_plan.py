"""The GEMM's plan of a product (host only), for tests that pin a tile shape."""
import ctypes as ct


def gemm_plan(sq, Mg, Ng, K, splits=1, ext=False):
    """(tile rows, tile columns, output rows of the first of two launches or 0); ext: with
    appended fold windows.  Tile 0 x 0: the register-staged kernel."""
    bm, bn, rows = ct.c_int32(0), ct.c_int32(0), ct.c_int64(0)
    sq.load().sq_internal_gemm_plan(ct.c_int64(Mg), ct.c_int64(Ng), ct.c_int64(K), ct.c_int32(splits), ct.c_int32(ext),
                                    ct.byref(bm), ct.byref(bn), ct.byref(rows))
    return bm.value, bn.value, rows.value
