"""The binding's two routes into the library, the call extension for plain integers and ctypes for
everything else: both reach the same entry point, and what ctypes refuses stays refused."""
import ctypes
from ctypes import c_void_p

import pytest

import paper_2406_09425_amd as S

DESC = S.ConvDesc(1, 14, 14, 64, 64, 3, 3, 1, 1, S.SGPRS_BF16, 1)


class Small(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int)]


class Sub(S.ConvDesc):
    pass


def conv(desc, p=16, pool=None, partition=0, ws_bytes=0):
    S.sgprs_conv2d(desc, p, p, p, p, None, p, None, ws_bytes, pool, partition)


def test_conv2d_takes_a_conv_desc_and_nothing_else():
    for bad in (Small(1), ctypes.pointer(DESC), (ctypes.c_int * 11)(), ctypes.byref(DESC), 16, None):
        with pytest.raises((ctypes.ArgumentError, TypeError)):
            conv(bad)
    for good in (DESC, Sub(1, 14, 14, 64, 64, 3, 3, 1, 1, S.SGPRS_BF16, 1)):
        with pytest.raises(S.SgprsError, match="pool is NULL"):
            conv(good)


def dead_task():
    t = S.Task.__new__(S.Task)
    t.handle = t.address = None
    return t


CALLS = {
    "conv2d": (conv, "pool is NULL", lambda p, i: (DESC, p, None, i)),
    "maxpool2d": (S.sgprs_maxpool2d, "pool is NULL", lambda p, i: (1, 1, 14, 14, 64, p, p, None, i)),
    "bn_relu": (S.sgprs_bn_relu, "pool is NULL", lambda p, i: (1, 8, 64, p, p, p, p, None, i)),
    "add_relu": (S.sgprs_add_relu, "pool is NULL", lambda p, i: (1, 64, p, p, p, True, None, i)),
    "avgpool_fc": (S.sgprs_avgpool_fc, "pool is NULL", lambda p, i: (1, 1, 49, 512, 1000, p, p, None, p, p, None, i)),
    "avgpool_fc_static": (S.sgprs_avgpool_fc_static, "pool is NULL", lambda p, i: (1, 1, 49, 512, 1000, p, p, None, p, None, i)),
    "global_avgpool": (S.sgprs_global_avgpool, "pool is NULL", lambda p, i: (1, 1, 49, 512, p, p, None, i)),
    "stage_run": (lambda *a: dead_task().stage_run(*a), "task is NULL", lambda p, i: (0, 1, p, p, None, i)),
    "task_run": (lambda *a: dead_task().run(*a), "task is NULL", lambda p, i: (1, p, p, None, i)),
}


@pytest.mark.parametrize("name", CALLS)
def test_both_routes_reach_the_entry_point(name, monkeypatch):
    call, text, args = CALLS[name]
    calls, native = [], S.binding._calls()

    class Spy:
        def __getattr__(self, attr):
            def f(*a):
                rc = getattr(native, attr)(*a)
                calls.append(rc)
                return rc
            return f
    monkeypatch.setattr(S.binding, "_native", Spy())
    with pytest.raises(S.SgprsError, match=text):
        call(*args(16, 0))
    assert len(calls) == 1 and calls[0] < 0            # the extension made the call
    calls.clear()
    with pytest.raises(S.SgprsError, match=text):
        call(*args(c_void_p(16), 0))
    assert calls == [None]                             # a c_void_p is for ctypes
    for bad in (args(16, 1.5), args(1.5, 0)):
        with pytest.raises(ctypes.ArgumentError):
            call(*bad)
