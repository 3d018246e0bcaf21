"""Which kernels a layer call runs: the library's own plan (slim_host.h), read through its C++ symbol."""
import ctypes

from paper_2608_24070_amd import slim

_int, _i64, _size = ctypes.c_int, ctypes.c_int64, ctypes.c_size_t


class Plan(ctypes.Structure):
    _fields_ = [("ad_tiles_m", _int), ("ad_tiles_j", _int), ("ad_split", _int), ("ad_tn", ctypes.c_bool),
                ("ad_wide", ctypes.c_bool), ("ad_slice", _i64), ("ad_sub", _int), ("ad_jblocks", _i64),
                ("mid", ctypes.c_bool), ("decode", ctypes.c_bool), ("dec_fm", _int), ("dec_g", _int),
                ("sp_rows_tile", _int), ("sp_cols_tile", _int), ("sp_row_tiles", _i64), ("sp_col_tiles", _i64),
                ("sp_split", _int), ("dec_units", _int), ("sp_blocks", _i64), ("sp_chunks_per_split", _i64),
                ("lds_bytes", _size), ("scaled", ctypes.c_bool)] + [
                    (n, _size) for n in ("off_counters", "n_counters", "off_t", "off_tpart", "off_ypart", "off_x16",
                                         "off_rowinv", "off_pb", "total", "query", "off_q16", "off_p16")]


def plan(kind, m, n, k, r, ws_bytes=1 << 62):
    """The plan of a "fwd" or "dx" call with a workspace of ws_bytes."""
    f = slim.lib()._Z14slim_make_planbllllmP8SlimPlan
    f.argtypes = [ctypes.c_bool, _i64, _i64, _i64, _i64, _size, ctypes.POINTER(Plan)]
    p = Plan()
    assert f(kind == "dx", m, n, k, r, ws_bytes, ctypes.byref(p)) == slim.SLIM_OK
    # the layout above is the library's: its workspace query agrees
    query = slim.slim_bwd_dx_workspace if kind == "dx" else slim.slim_linear_workspace
    assert p.query == query(m, n, k, r)
    return p
