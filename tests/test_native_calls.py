"""The compiled marshalling of the per-step calls hands the C entry points what
ctypes and plain Python conversions hand them, for every form of an argument; and so
does what takes its place under a Python that it is not built for."""
import ctypes
import os
import shutil
import subprocess
import sys
import sysconfig
from collections import namedtuple

import numpy as np
import pytest
import torch

from paper_2606_00539_amd import binding as B

P, I32, I64, D = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_double
SIGNATURES = {
    "gnmr_step": (P, D, D, P, P), "gnmr_step_from_norms": (P, P, D, D, P),
    "gnmr_step_from_partials": (P, P, D, D, P), "gnmr_sumsq": (P, P, P, P),
    "gnmr_actuate": (P, P, I32, I32, P),
    "gnmr_actuate_matrix": (P, P, I64, I32, P, I32, I32, I32, P),
    "gnmr_wgrad_sumsq": (P, P, P, I64, I32, I32, P, P),
    "gnmr_wgrad_sumsq_batched": (P, I32, P, P),
}


class Buffer:
    def __init__(self, p):
        self.p = p

    def data_ptr(self):
        if isinstance(self.p, Exception):
            raise self.p
        return self.p


class Stream:
    cuda_stream = 0x7F0000001230


class Rows:
    """A sequence that is neither a tuple nor a list."""

    def __init__(self, *v):
        self.v = v

    def __getitem__(self, k):
        return self.v[k]

    def __len__(self):
        return len(self.v)


Problem = namedtuple("Problem", "dy x dw tokens outf inf acc")


def recording():
    """Binds the module to functions that record what they are given; -7 is
    the status they return."""
    keep, got = [], []

    def record(name):
        def f(*a):
            a = [x if x is not None or t is not P else 0 for x, t in zip(a, SIGNATURES[name])]
            lists = []
            if name in ("gnmr_step", "gnmr_sumsq"):
                k = 3 if name == "gnmr_step" else 1
                if a[k]:
                    lists = [v or 0 for v in (ctypes.c_void_p * got.count).from_address(a[k])]
                a[k] = bool(a[k])
            if name == "gnmr_wgrad_sumsq_batched":
                ps = (B.gnmr_wgrad_problem * a[1]).from_address(a[0])
                lists = [tuple(getattr(p, n) or 0 for n, _ in p._fields_) for p in ps]
                a[0] = bool(a[0])
            got.append((a, lists))
            return -7
        return f

    class Seen(list):
        count = 0
    got = Seen()
    fns = {}
    for name, args in SIGNATURES.items():
        fns[name] = ctypes.CFUNCTYPE(ctypes.c_int, *args)(record(name))
    keep.append(fns)
    return keep, got, {n: ctypes.cast(f, P).value for n, f in fns.items()}


@pytest.fixture
def seen():
    calls = B._native()
    keep, got, addresses = recording()
    calls.bind(addresses)
    try:
        yield calls, got
    finally:
        calls.bind({n: ctypes.cast(getattr(B.load_library(), n), P).value for n in B._PER_STEP})


@pytest.fixture(params=["compiled", "ctypes"])
def either(request):
    if request.param == "compiled":
        yield request.getfixturevalue("seen")
    else:
        keep, got, addresses = recording()
        calls = B._CtypesCalls(B.load_library())
        calls.bind(B.load_library(), addresses)
        yield calls, got


def pointer(p):
    return p.data_ptr() if hasattr(p, "data_ptr") else int(p)


def stream_of(s):
    return 0 if s is None else int(getattr(s, "cuda_stream", s))


X = torch.zeros(4)
POINTERS = [X, X[1:], Buffer(0xFEDCBA9876543210), 4096, np.int64(8192), np.uint64(2**63 + 16), 0,
            True, 3.0, "65536"]
STREAMS = [None, 0, 77, Stream(), np.int64(5)]
HANDLES = [None, ctypes.c_void_p(), ctypes.c_void_p(0x7FFFFFFFFFF0), 1234]
WHOLE = [5, np.int32(7), 2**31 + 3, -1, 9.9, 2**40 + 2]
FLOATS = [1.5, 2, np.float32(0.25), torch.tensor(0.5), "1e-3", float("nan")]


def word(v, bits):
    return ctypes.c_int32(int(v)).value if bits == 32 else ctypes.c_int64(int(v)).value


def handle(h):
    return (h.value if isinstance(h, ctypes.c_void_p) else h) or 0


def u64(v):
    return v & (2**64 - 1)


def same(a, b):
    return a == b or (a != a and b != b)


@pytest.mark.parametrize("k", range(10))
def test_every_form_of_an_argument(either, k):
    calls, got = either
    p, q, r = (POINTERS[(k + j) % len(POINTERS)] for j in (0, 3, 5))
    s, h = STREAMS[k % len(STREAMS)], HANDLES[k % len(HANDLES)]
    w, v = WHOLE[k % len(WHOLE)], WHOLE[(k + 1) % len(WHOLE)]
    a, b = FLOATS[k % len(FLOATS)], FLOATS[(k + 2) % len(FLOATS)]
    pp, qq, rr, ss, hh = u64(pointer(p)), u64(pointer(q)), u64(pointer(r)), stream_of(s), handle(h)
    want = [[hh, pp, float(a), float(b), ss], [hh, pp, float(a), float(b), ss],
            [hh, pp, word(w, 32), word(v, 32), ss],
            [pp, qq, word(w, 64), word(v, 32), rr, word(v, 32), word(w, 32), word(v, 32), ss],
            [pp, qq, rr, word(w, 64), word(v, 32), word(w, 32), qq, ss]]
    status = [calls.step_from_norms(h, p, a, b, s), calls.step_from_partials(h, p, a, b, s),
              calls.actuate(h, p, w, v, s), calls.actuate_matrix(p, q, w, v, r, v, w, v, s),
              calls.wgrad_sumsq(p, q, r, w, v, w, q, s)]
    assert status == [-7] * 5
    for (args, _), ref in zip(got, want):
        assert all(same(x, y) for x, y in zip(args, ref)), (args, ref)


# around the 256 pointers that are marshalled on the stack
@pytest.mark.parametrize("n", [0, 1, 10, 255, 256, 257, 5000])
@pytest.mark.parametrize("form", [list, tuple, iter, np.array])
def test_pointer_lists(either, n, form):
    calls, got = either
    got.count = max(n, 1)
    vals = [POINTERS[i % len(POINTERS)] for i in range(n)]
    if form is np.array:
        vals = [4096 + 16 * i for i in range(n)]
    want = [u64(pointer(p)) for p in vals] or [0]
    assert calls.step(5, 1.0, 2.0, form(vals), 9) == calls.sumsq(5, form(vals), X, None) == -7
    assert got[0] == ([5, 1.0, 2.0, True, 9], want)
    assert got[1] == ([5, True, X.data_ptr(), 0], want)
    assert calls.step(5, 1.0, 2.0, None, 9) == -7 and got[2] == ([5, 1.0, 2.0, False, 9], [])


def test_problems(either):
    calls, got = either
    ps = [(X, 4096, Buffer(64), 10, 20, 30), [X, X, X, 1.9, 2**32 + 8, 16, True],
          Problem(16, 32, 48, 2**40, 8, 8, 1), Rows(16, 32, 48, 5, 6, 7),
          Rows(16, 32, 48, 5, 6, 7, 1), (16, 32, 48, 1, 2, 3, 1, "more")] * 9
    want = []
    for p in ps:
        a, b, c, t, o, i = p[:6]
        want.append((pointer(a), pointer(b), pointer(c), word(t, 64), word(o, 32), word(i, 32),
                     int(p[6]) if len(p) > 6 else 0, 0))
    for form in (list, tuple, iter):
        assert calls.wgrad_sumsq_batched(form(ps), X, Stream()) == -7
        assert got.pop() == ([True, len(ps), X.data_ptr(), Stream.cuda_stream], want)
    assert calls.wgrad_sumsq_batched([], X, None) == -7
    assert got.pop() == ([True, 0, X.data_ptr(), 0], [])


@pytest.mark.parametrize("bad", [None, "x", object(), [1], Buffer("7"), Buffer(KeyError("mine")),
                                 Buffer(AttributeError("mine"))])
def test_what_is_no_pointer_is_refused(seen, bad):
    calls, got = seen
    kind = type(bad.p) if isinstance(bad, Buffer) and isinstance(bad.p, Exception) else \
        (TypeError, ValueError)
    for call in (lambda: calls.step(5, 1.0, 2.0, [X, bad], None),
                 lambda: calls.step(5, 1.0, 2.0, [X] * 300 + [bad], None),
                 lambda: calls.actuate(5, bad, 1, 0, None),
                 lambda: calls.actuate_matrix(X, X, 1, 8, bad, 0, 1, 0, None),
                 lambda: calls.wgrad_sumsq(X, X, X, 1, 8, 8, bad, None),
                 lambda: calls.wgrad_sumsq_batched([(X, X, bad, 1, 8, 8)], X, None)):
        with pytest.raises(kind):
            call()
    assert not got


@pytest.mark.parametrize("call", [
    lambda c: c.step("ctx", 1.0, 2.0, None, None), lambda c: c.step(5, None, 2.0, None, None),
    lambda c: c.step(5, 1.0, 2.0, 7, None), lambda c: c.step(5, 1.0, 2.0, None, "s"),
    lambda c: c.step(5, 1.0, 2.0, None), lambda c: c.actuate(5, X, None, 0, None),
    lambda c: c.actuate_matrix(X, X, [1], 8, X, 0, 1, 0, None),
    lambda c: c.wgrad_sumsq_batched([(X, X, X, 1, 8)], X, None),
    lambda c: c.wgrad_sumsq_batched([iter((X, X, X, 1, 8, 8))], X, None),
    lambda c: c.wgrad_sumsq_batched([(X, X, X, 1, 8, 8, None)], X, None),
    lambda c: c.wgrad_sumsq_batched(X.data_ptr(), X, None)])
def test_other_refusals(seen, call):
    calls, got = seen
    with pytest.raises((TypeError, ValueError, AttributeError)):
        call(calls)
    assert not got


def test_the_module_is_the_compiled_one():
    assert B._native().__file__.endswith(sysconfig.get_config_var("EXT_SUFFIX"))


def test_another_python_does_not_load_the_module(tmp_path):
    """The package in a copy whose module is that of another Python: it loads, says
    so, and calls through ctypes."""
    pkg = os.path.dirname(B.__file__)
    ext = sysconfig.get_config_var("EXT_SUFFIX")
    copy = shutil.copytree(pkg, tmp_path / "paper_2606_00539_amd",
                           ignore=shutil.ignore_patterns("__pycache__", "csrc"))
    os.rename(copy / ("_calls" + ext), copy / "_calls.cpython-399-x86_64-linux-gnu.so")
    code = """
import warnings
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    import paper_2606_00539_amd as g
    from paper_2606_00539_amd import binding as B
    assert type(B._native()).__name__ == "_CtypesCalls"
    assert any("not built for this Python" in str(w.message) for w in seen)
for call in (lambda: g.gnmr_step(None, 1.0, 1.0), lambda: g.gnmr_actuate(None, 4096, 1, 0),
             lambda: g.gnmr_wgrad_sumsq(4096, 8192, 16384, 16, 12, 128, 32768)):
    try:
        call()
        raise SystemExit("accepted")
    except g.GnmrError as e:
        assert e.status == g.binding.GNMR_E_INVALID, e
print("good")
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True,
                       env={k: v for k, v in os.environ.items() if k != "GNMR_LIBRARY"}, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "good", r.stdout + r.stderr
