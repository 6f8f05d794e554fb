"""The library's choice of a pooled lookup's kernel (include/eb_route.h), on the host."""
import ctypes

from paper_2512_05831_amd import eb

PLAIN, TEAM, WAVE = 0, 1, 2


class Call(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("D", "dtype", "mode", "table_align", "out_align", "offsets_align")] + \
               [(n, ctypes.c_int64) for n in ("T", "B", "nnz", "table_rows", "local_rows")]


class Route(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("kernel", "chunk_bytes", "lanes", "chunks", "small_batch", "narrow",
                                              "non_temporal", "xcd_runs", "split")]


def route(D, dtype, T, B, ids, rows, local=None, hint=False, align=16, out_align=16):
    """The route of T x B bags of `ids` ids on average."""
    call = Call(D=D, dtype=dtype, mode=eb.EB_HINT_STREAM_ROWS if hint else 0, table_align=align, out_align=out_align,
                offsets_align=16, T=T, B=B, nnz=round(T * B * ids), table_rows=rows,
                local_rows=rows if local is None else local)
    r = Route()
    assert eb.library().eb_gather_route(ctypes.byref(call), ctypes.byref(r)) == 0
    return r
