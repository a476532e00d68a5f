"""Argument marshalling of the binding (no GPU): the cheap conversions give the
same tables as numpy's, for every form that callers pass."""
import ctypes

import numpy as np
import pytest

from paper_2608_23429_amd import _binding as B


def _read(p, ctype, n):
    # byref() and pointer objects both pass as arguments; read them back alike
    return list((ctype * n).from_address(ctypes.cast(p, ctypes.c_void_p).value)) if n else []


@pytest.mark.parametrize("values", [
    [], [0], [3, -1, 1 << 62], [np.int64(7), 5], (1, 2, 3), [True, 2], [1.0, 2.0],
    np.arange(5), np.arange(6, dtype=np.int32), np.arange(8)[::2]])
def test_int64_tables(values):
    p, n = B._i64ptr(values)
    want = np.ascontiguousarray(values, dtype=np.int64).reshape(-1)
    assert n == want.size
    assert _read(p, ctypes.c_int64, n) == want.tolist()


@pytest.mark.parametrize("values", [[1 << 63], ["a"], [None]])
def test_int64_tables_refuse_what_numpy_refuses(values):
    with pytest.raises((OverflowError, TypeError, ValueError)) as want:
        np.ascontiguousarray(values, dtype=np.int64)
    with pytest.raises(want.type):
        B._i64ptr(values)


@pytest.mark.parametrize("ptrs", [
    [], [0], [1 << 47, 16], (64, 128), [np.uint64(4096), 32], [48.0], np.array([16, 32])])
def test_address_tables(ptrs):
    p = B._voidp_array(ptrs)
    want = [int(v) for v in ptrs]
    assert _read(p, ctypes.c_uint64, len(want)) == want


def test_fp64_pointers_and_results():
    w = np.array([1.0, -2.5])
    ro = w.copy()
    ro.flags.writeable = False
    for a in (w, ro):
        assert _read(B._dptr(a), ctypes.c_double, 2) == [1.0, -2.5]
    buf = (ctypes.c_double * 4)(1.0, 2.0, 3.0, 4.0)
    out = B._doubles(buf, 3)
    assert out.dtype == np.float64 and out.tolist() == [1.0, 2.0, 3.0] and out.flags.writeable
    assert B._doubles(buf, 0).size == 0
    # a frozen or strided weight row goes in like any other
    x = np.array([0.0, 1.0, 2.0])
    x.flags.writeable = False
    want = B.cheb_precompute_weights([0.0, 1.0, 2.0], [3.0])
    assert np.array_equal(B.cheb_precompute_weights(x, np.array([3.0, 9.0])[::2]), want)


class _Writes:
    """Stands for the library: every call succeeds and fills the weights."""

    def __getattr__(self, name):
        def call(*args):
            rows = args[-1]
            for i in range(len(rows)):
                rows[i] = float(i)
            return B.CHEB_OK
        return call


@pytest.mark.parametrize("n_slots", [0, 1, B.CHEB_MAX_SLOTS, B.CHEB_MAX_SLOTS + 1, 40])
def test_weights_clipped_to_what_the_library_holds(monkeypatch, n_slots):
    """A history size past the largest gives what is there, not an error after
    the launch has gone out."""
    monkeypatch.setattr(B, "LIB", _Writes())
    most = np.arange(float(B.CHEB_MAX_SLOTS * B.CHEB_MAX_OUTPUTS))
    assert np.array_equal(B.cheb_extrapolate_at(0, 0.5, 0, n_slots=n_slots),
                          most[:min(n_slots, B.CHEB_MAX_SLOTS)])
    if n_slots <= B.CHEB_MAX_SLOTS + 1:        # the rows are packed
        assert np.array_equal(B.cheb_extrapolate_at_multi(0, [0.5, 0.6], [0, 0], n_slots=n_slots),
                              most[:2 * n_slots].reshape(2, n_slots))
