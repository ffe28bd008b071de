"""The native calls of the binding against ctypes: every entry point that has one, at a C function that
notes its arguments, with plain values at the ends of their ranges and with what only ctypes converts."""
import ctypes
import math
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2208_14228_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

B.lib()
native = pytest.importorskip("paper_2208_14228_amd._pycall")


def _probe(name):
    """(native call, ctypes call, notes): both at the same C function, which returns -4."""
    types = B._SIGS[name][1]
    # pointers to arrays travel as addresses
    plain = [ctypes.c_void_p if issubclass(t, ctypes._Pointer) else t for t in types]
    notes = []
    proto = ctypes.CFUNCTYPE(ctypes.c_int, *plain)
    target = proto(lambda *a: notes.append(a) or -4)
    address = ctypes.cast(target, ctypes.c_void_p).value
    general = ctypes.CFUNCTYPE(ctypes.c_int, *plain)(address)
    seen = []
    call = native.bind(name, address, lambda *a, **k: seen.append((a, k)) or general(*a, **k))
    return call, general, plain, notes, seen, target


def _ends(t):
    if t is ctypes.c_void_p:
        return [None, 0, 1, 1 << 47, (1 << 64) - 1]
    if t in (ctypes.c_uint32, ctypes.c_uint64):
        return [0, 1, (1 << 8 * ctypes.sizeof(t)) - 1]
    return [0.0, -0.0, 0.1, 1e300, -1e-320, math.inf, math.nan]


@pytest.mark.parametrize("name", native.NAMES)
def test_same_arguments_as_ctypes(name):
    call, general, types, notes, seen, _ = _probe(name)
    base = [_ends(t)[1] if i else 12345 for i, t in enumerate(types)]
    for i, t in enumerate(types):
        for v in _ends(t):
            args = base[:i] + [v] + base[i + 1:]
            notes.clear()
            assert call(*args) == -4 and general(*args) == -4
            assert len(notes) == 2 and repr(notes[0]) == repr(notes[1]), (i, v)
    assert not seen                                     # none of these needs the general function


@pytest.mark.parametrize("name", native.NAMES)
def test_the_rest_is_left_to_the_general_function(name):
    call, general, types, notes, seen, target = _probe(name)
    base = [_ends(t)[1] if i else 12345 for i, t in enumerate(types)]
    for i, t in enumerate(types):
        odd = [np.int64(3), "3", -1, True, 1 << 64] + ([3] if t in (ctypes.c_float, ctypes.c_double) else [1.0])
        for v in odd + ([1 << 32] if t is ctypes.c_uint32 else []):
            args = base[:i] + [v] + base[i + 1:]
            notes.clear()
            seen.clear()
            results = []
            for f in (call, general):
                try:
                    results.append((f(*args), None))
                except Exception as e:
                    results.append((None, type(e)))
            assert len(seen) == 1 and results[0] == results[1], (i, v)
            assert len(notes) in (0, 2) and (not notes or repr(notes[0]) == repr(notes[1])), (i, v)
    notes.clear()
    call = native.bind(name, ctypes.cast(target, ctypes.c_void_p).value, lambda *a, **k: (a, k))
    for args, kw in [(base[:-1], {}), (base + [0], {}), (base, {"x": 1}), (base[:-1], {"x": 1}), ([], {})]:
        assert call(*args, **kw) == (tuple(args), kw)
    assert not notes


def test_bound_calls_keep_names_defaults_and_status():
    import inspect
    for name in native.NAMES:
        if name == "es_est_boundary":
            continue
        f = getattr(B, name)
        assert f.__name__ == name and inspect.signature(f) == inspect.signature(f.__wrapped__)
        assert f.__wrapped__.__module__ == B.__name__
    assert B.es_bn_batch_stats(None, 0, 1, 1, None, None, None, 0) == B.ES_EINVAL
    assert B.es_stage_fence(h=None) == B.ES_EINVAL
    with pytest.raises(ValueError):
        native.bind("es_init", 1, len)


@pytest.mark.parametrize("which", ["b", "g"])
def test_an_array_put_in_the_place_of_a_marshalled_one_is_used(monkeypatch, which):
    notes = []
    monkeypatch.setattr(B, "_boundary", lambda *a: notes.append(a) or -7)
    proto = ctypes.CFUNCTYPE(ctypes.c_int, *B._SIGS["es_est_boundary"][1])
    general = proto(lambda h, out, into, n, b, g: notes.append((h, out, into, n, b[0], g[0])) or -8)
    class Library:
        es_est_boundary = general
    monkeypatch.setattr(B, "lib", lambda: Library)
    m = B.Marshalled([3], [64])
    at = ctypes.addressof(m.b), ctypes.addressof(m.g)
    assert B.es_est_boundary_m(5, 0, None, m) == -7 and notes == [(5, 0, B.ES_NO_EST, 1, *at)]
    setattr(m, which, (ctypes.c_uint32 * 1)(9) if which == "b" else (ctypes.c_void_p * 1)(128))
    notes.clear()
    assert B.es_est_boundary_m(5, 0, 2, m) == -8
    assert notes == [(5, 0, 2, 1, *((9, 64) if which == "b" else (3, 128)))]


def test_a_module_built_from_other_sources_is_not_used(monkeypatch):
    import types

    import paper_2208_14228_amd as package
    for attrs in ({"SOURCE_HASH": "0" * 16}, {}):
        stale = types.SimpleNamespace(NAMES=native.NAMES, bind=lambda *a: pytest.fail("a stale module is bound"), **attrs)
        monkeypatch.setattr(package, "_pycall", stale)
        with pytest.warns(RuntimeWarning, match="built from other sources"):
            B._bind_native(B.lib())


def test_a_function_put_in_before_the_library_is_loaded_stays():
    code = """
import functools
from paper_2208_14228_amd import binding as B
seen = []
plain = lambda h: seen.append(h) or -9
@functools.wraps(B.es_ctx_save)
def traced(h, est): seen.append(est); return B.es_ctx_save.__wrapped__(h, est)
B.es_stage_fence, B.es_ctx_save = plain, traced
B.lib()
assert B.es_stage_fence is plain and B.es_stage_fence(None) == -9
assert B.es_ctx_save is traced and B.es_ctx_save(None, 7) == B.ES_EINVAL and seen == [None, 7]
assert type(B.es_ctx_restore).__name__ == "Bound" and B.es_ctx_restore(None, 0) == B.ES_EINVAL
"""
    subprocess.run([sys.executable, "-c", code], check=True, timeout=120, cwd=ROOT)
