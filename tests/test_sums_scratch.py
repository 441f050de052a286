"""Who waits for whom among overlapping calls with sums (CPU: the library's host
code against a runtime that launches nothing)."""
import ctypes
import threading

from launches import recorder  # noqa: F401  (fixture)
from paper_1402_5487_amd import _plbm


def _call(rec, entry, stream, out):
    d = _plbm.desc_default(2, 300, 200, 1.5, "f64")
    s = (ctypes.c_double * 4)()
    out.append(getattr(rec.lib, entry)(ctypes.byref(d), 0x1000, 0x2000, 3, s, stream))


def _overlap(rec, first, second):
    """Whether `second` returns while `first`, on another stream, still runs."""
    rec.lib.rec_busy.argtypes = [ctypes.c_void_p]
    done = []
    rec.lib.rec_busy(0x77)
    a = threading.Thread(target=_call, args=(rec, first, 0x77, done))
    a.start()
    rec.lib.rec_await()
    b = threading.Thread(target=_call, args=(rec, second, 0x88, done))
    b.start()
    b.join(timeout=5)
    returned = not b.is_alive()
    rec.lib.rec_busy(None)
    a.join(timeout=60)
    b.join(timeout=60)
    assert done == [_plbm.PLBM_OK] * 2
    return returned


def test_a_call_without_allocation_does_not_wait_for_plbm_step(recorder):  # noqa: F811
    assert _overlap(recorder, "plbm_step", "plbm_step_noalloc")


def test_other_calls_wait_for_none(recorder):  # noqa: F811
    assert _overlap(recorder, "plbm_step", "plbm_step")
    assert _overlap(recorder, "plbm_step_noalloc", "plbm_step")


def test_calls_without_allocation_take_turns(recorder):  # noqa: F811
    assert not _overlap(recorder, "plbm_step_noalloc", "plbm_step_noalloc")
