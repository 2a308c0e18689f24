"""CPU: the native argument conversion of the binding's launching calls (every
call here ends in the library's own argument checks, before any device work)."""
import re
import sys
import types

import numpy as np
import pytest
import torch

from paper_2511_20982_amd import attn as A


class FakeDevice:
    """Stands for a device tensor: an address and nothing else."""

    def data_ptr(self):
        return 0x7F0000000000


P = FakeDevice()
CU = np.array([0, 4], np.int32)


def status(fn, *args, **kw):
    try:
        fn(*args, stream=0, **kw)
    except A.DopdError as e:
        return e.status
    return A.DOPD_OK


def prefill(shape=None, q=P, lse=None, cu_host=CU, n=1, **kw):
    shape = A.make_shape(8, 2, 128) if shape is None else shape
    return status(A.dopd_prefill_attn, shape, q, P, P, P, lse, P, cu_host, n, **kw)


def test_statuses_come_back():
    assert prefill(A.make_shape(6, 4, 128)) == A.DOPD_ERR_INVALID_SHAPE
    assert prefill(A.make_shape(8, 2, 96)) == A.DOPD_ERR_UNSUPPORTED
    assert prefill(q=None) == A.DOPD_ERR_NULL_POINTER
    assert prefill(cu_host=None) == A.DOPD_ERR_NULL_POINTER
    assert prefill(cu_host=[1, 4]) == A.DOPD_ERR_INVALID_SHAPE       # cu[0] != 0, read through the pointer
    assert prefill(cu_host=np.array([0, 4, 2], np.int64), n=np.int64(2)) == A.DOPD_ERR_INVALID_SHAPE
    assert prefill(cu_host=[0, 0]) == A.DOPD_OK                      # all empty
    assert prefill(n=0) == A.DOPD_OK
    shape = A.make_shape(8, 2, 128)
    assert status(A.dopd_decode_attn, shape, P, P, P, 10, P, 1, P, [40], 1, 0, P, None, P,
                  workspace_bytes=1 << 40) == A.DOPD_ERR_INVALID_SHAPE   # more pages than the table's row
    assert status(A.dopd_decode_attn, shape, P, P, P, 10, P, 1024, P, [40], 1, 0, P, None, P,
                  workspace_bytes=64) == A.DOPD_ERR_WORKSPACE_TOO_SMALL
    assert status(A.dopd_kv_write, shape, P, P, P, P, 10, P, 4, P, P, 0, 0) == A.DOPD_OK


def test_what_is_no_device_pointer_is_refused():
    with pytest.raises(AttributeError):
        prefill(q=np.zeros(4, np.float32))
    with pytest.raises(AttributeError):
        prefill(lse=5)
    with pytest.raises(TypeError):
        prefill(shape=0)
    with pytest.raises((TypeError, ValueError)):
        prefill(n="many")
    t = torch.zeros(4)
    assert prefill(lse=t, cu_host=[0, 0]) == A.DOPD_OK


@pytest.mark.parametrize("shape", [b"", b"\0" * 24, np.array([8, 2, 128, 16, 0, 0], np.int32), bytearray(100), None])
def test_only_a_shape_is_a_shape(shape):
    """Whatever exports a buffer is refused before its bytes are read."""
    with pytest.raises(TypeError):
        A.dopd_prefill_attn(shape, P, P, P, P, None, P, CU, 1, stream=0)
    with pytest.raises(TypeError):
        A.dopd_decode_attn_noalloc(shape, P, P, P, 10, P, 1024, P, [40], 1, 0, P, None, stream=0)


def test_a_class_derived_from_shape_is_one():
    class Named(A.Shape):
        pass

    assert prefill(Named(6, 4, 128, 16, A.DOPD_BF16, 1.0)) == A.DOPD_ERR_INVALID_SHAPE


def test_every_launching_entry_point_is_bound():
    A.lib()
    m = A._calls()
    bound = [f for f in dir(m) if f.startswith("dopd_")]
    host_only = {f for f in A.EXPORTS if re.search(r"_size$|_host$|status_string|last_hip_error", f)}
    assert set(bound) == set(A.EXPORTS) - host_only
    for f in bound:
        with pytest.raises(TypeError):
            getattr(m, f)(1, 2)


MODULE = "paper_2511_20982_amd._marshal"


def replace_module(monkeypatch, m):
    """The module the binding finds at its next launching call (None: none)."""
    import paper_2511_20982_amd as package
    monkeypatch.setattr(A, "_CALLS", None)
    monkeypatch.delattr(package, "_marshal", raising=False)
    monkeypatch.setitem(sys.modules, MODULE, m)


def test_host_only_calls_need_no_module(monkeypatch):
    replace_module(monkeypatch, None)
    shape = A.make_shape(8, 2, 128)
    assert A.dopd_decode_workspace_size(shape, np.array([40], np.int32), 1) > 0
    assert A.status_string(A.DOPD_OK)
    with pytest.raises(RuntimeError, match="not built.*build"):
        prefill()


def test_a_module_of_other_sources_is_refused(monkeypatch):
    real = A._calls()
    other = types.ModuleType(MODULE)
    for f in dir(real):
        setattr(other, f, getattr(real, f))
    changed = lambda *a: 0  # noqa: E731
    changed.__doc__ = A.LAUNCHES["dopd_kv_write"] + "p"
    other.dopd_kv_write = changed
    replace_module(monkeypatch, other)
    with pytest.raises(RuntimeError, match="other sources"):
        prefill()


def test_the_tables_name_every_launching_entry_point():
    host_only = {f for f in A.EXPORTS if re.search(r"_size$|_host$|status_string|last_hip_error", f)}
    assert set(A.LAUNCHES) == set(A.EXPORTS) - host_only
