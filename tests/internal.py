"""The library's inner decisions, as its tests look at them (csrc/difa_testing.h)."""
import ctypes

import numpy as np

from paper_2503_22796_amd import binding as B

_vp, _i32, _i32p = ctypes.c_void_p, ctypes.c_int32, ctypes.POINTER(ctypes.c_int32)
_L = B.lib
_L.difa_testing_records.argtypes = [_i32, _i32, _vp, _vp, _i32, _i32, _i32, _i32, ctypes.c_uint32, _vp, _i32, _i32p]
_L.difa_testing_schedule.argtypes = [_vp, _i32, _i32, _i32, _i32, _vp, _vp, _vp, _i32, _vp, _i32p, _vp, _i32, _i32p, _i32p, _i32p]
_L.difa_testing_record_rows.argtypes = [_i32, _i32, _i32, _vp, _vp, _i32, _i32, ctypes.c_uint32, _i32]
_L.difa_testing_trial.argtypes = [_i32, _vp, _i32, _vp, _i32, _vp, _vp, _vp]
_L.difa_testing_victim.argtypes = [_i32, _vp, _vp, _vp]
_L.difa_testing_trial.restype = None
_L.difa_testing_copy_chunks.argtypes = [ctypes.c_int64, _i32, _i32, _i32, _i32]
_L.difa_testing_schedule_memory.argtypes = [_i32, _i32, _i32, _i32, _i32, _vp, _vp, _i32p]
_L.difa_testing_schedule_memory.restype = None
_L.difa_testing_force_rows.argtypes = [_vp, _i32]
_L.difa_testing_last_call.argtypes = [_vp] + [_i32p] * 5
_L.difa_testing_last_call.restype = None


def _i32a(a):
    return np.ascontiguousarray(np.asarray(a, dtype=np.int32))


def _dtype(struct):
    return np.dtype([(n, np.int32) for n, _ in struct._fields_])


def records(batch, head_plan, window, n_text, n_img, rows, head_dim, flags=0):
    """The records of a layer as the bf16 kernel gets them, in the scheduler's order."""
    hp, win, n = _i32a(head_plan), _i32a(window), _i32(0)
    args = (batch, len(hp), hp.ctypes.data, win.ctypes.data, n_text, n_img, rows, head_dim, flags)
    assert _L.difa_testing_records(*args, None, 0, ctypes.byref(n)) == B.DIFA_OK
    out = np.zeros(n.value, dtype=_dtype(B.difa_work_item_t))
    assert _L.difa_testing_records(*args, out.ctypes.data if len(out) else None, len(out), ctypes.byref(n)) == B.DIFA_OK
    return out


def schedule(items, head_dim, n_wg, n_xcd=8, speeds=None):
    """The library's own schedule of them: (segments, wg_begin, merges, scratch slots, die spans, plans with cuts looked at)."""
    segs = np.zeros(len(items) + 2 * n_wg, dtype=_dtype(B.difa_segment_t))
    merges = np.zeros(2 * n_wg, dtype=_dtype(B.difa_merge_item_t))
    wg_begin, span = np.zeros(n_wg + 1, np.int32), np.zeros(n_xcd, np.int64)
    n_segs, n_merges, n_slots, tried = (_i32(0) for _ in range(4))
    sp = None if speeds is None else np.ascontiguousarray(speeds, dtype=np.float64)
    assert sp is None or len(sp) == n_xcd
    st = _L.difa_testing_schedule(items.ctypes.data, len(items), head_dim, n_wg, n_xcd, sp.ctypes.data if sp is not None else None,
                                  span.ctypes.data, segs.ctypes.data, len(segs), wg_begin.ctypes.data, ctypes.byref(n_segs),
                                  merges.ctypes.data, len(merges), ctypes.byref(n_merges), ctypes.byref(n_slots), ctypes.byref(tried))
    assert st == B.DIFA_OK
    return segs[:n_segs.value], wg_begin, merges[:n_merges.value], n_slots.value, span, tried.value


def record_rows(batch, head_dim, head_plan, window, n_text, n_img, flags=0, n_cu=256):
    hp, win = _i32a(head_plan), _i32a(window)
    return _L.difa_testing_record_rows(batch, len(hp), head_dim, hp.ctypes.data, win.ctypes.data, n_text, n_img, flags, n_cu)


def trial(die_span, die_ticks, n_launches, capturing=None):
    """(version each launch runs, speeds each launch's schedule was made for) when version v takes die_ticks[v] on the dies and
    the launches in `capturing` are recorded into a graph."""
    cap = _i32a([i in (capturing or ()) for i in range(n_launches)])
    span = np.ascontiguousarray(die_span, dtype=np.int64)
    ticks = np.ascontiguousarray(die_ticks, dtype=np.float64)
    version, speeds = np.zeros(n_launches, np.int32), np.zeros((n_launches, len(span)))
    _L.difa_testing_trial(len(span), span.ctypes.data, len(ticks), ticks.ctypes.data, n_launches, cap.ctypes.data, version.ctypes.data, speeds.ctypes.data)
    return version, speeds


def victim(valid, held, stamp):
    v, h, s = _i32a(valid), _i32a(held), np.ascontiguousarray(stamp, dtype=np.int64)
    return _L.difa_testing_victim(len(v), v.ctypes.data, h.ctypes.data, s.ctypes.data)


def force_rows(plan, rows):
    assert _L.difa_testing_force_rows(plan, rows) == B.DIFA_OK


def last_call(plan):
    v = [_i32(0) for _ in range(5)]
    _L.difa_testing_last_call(plan, *[ctypes.byref(x) for x in v])
    return dict(zip(("rows", "n_wg", "grid", "n_pieces", "reports"), (x.value for x in v)))


def copy_chunks(n_tokens, head_dim, dtype, batch, n_copy):
    return _L.difa_testing_copy_chunks(n_tokens, head_dim, dtype, batch, n_copy)


def schedule_memory(batch, heads, dtype, max_tokens, n_cu=256):
    """(device bytes, pinned host bytes, resident schedules) of a plan object."""
    mem, n = np.zeros(2, np.int64), _i32(0)
    _L.difa_testing_schedule_memory(batch, heads, dtype, max_tokens, n_cu, mem[:1].ctypes.data, mem[1:].ctypes.data, ctypes.byref(n))
    return int(mem[0]), int(mem[1]), n.value
