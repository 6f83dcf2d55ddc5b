"""The native call behind Problem.run: what it hands to tf_variant_run for tensors, addresses, None and streams. A Python
callback stands in for tf_variant_run; no GPU."""
import ctypes as C
import os
import sysconfig
import threading

import numpy as np
import pytest
import torch

from paper_2512_09196_amd import build, tf

RUN = C.CFUNCTYPE(C.c_int32, C.c_void_p, C.c_int32, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p)


@pytest.fixture
def call():
    tf.lib()
    m, seen = tf._pycall, []
    cb = RUN(lambda *a: seen.append(a) or len(seen))
    m.bind_stream(None, None)
    m.bind(C.cast(cb, C.c_void_p).value, lambda: 77)
    yield m, seen
    m.bind_stream(None, None)
    m.bind(C.cast(tf.lib().tf_variant_run, C.c_void_p).value, tf._current_stream)


def test_arguments(call):
    m, seen = call
    t = torch.zeros(8)
    big = 2 ** 64 - 16                       # an address with its top bit set stays what it is
    assert m.run(5, 3, t, big, None, t[1:], 0, 1 << 40, 9) == 1
    assert m.run(0, -1, None, None, None, None, None, 0, None) == 2
    assert seen == [(5, 3, t.data_ptr(), big, None, t.data_ptr() + 4, None, 1 << 40, 9), (None, -1, None, None, None, None, None, 0, 77)]


def test_stream(call):
    m, seen = call

    class Stream:
        cuda_stream = 1234
    m.run(1, 0, 0, 0, 0, 0, 0, 0, Stream())
    m.bind_stream(lambda dev: 100 + dev, lambda: 2)
    m.run(1, 0, 0, 0, 0, 0, 0, 0, None)
    m.bind_stream(None, None)
    m.run(1, 0, 0, 0, 0, 0, 0, 0, None)
    assert [s[-1] for s in seen] == [1234, 102, 77]


def test_errors_reach_the_caller_and_nothing_runs(call):
    m, seen = call

    def broken(*a):
        raise RuntimeError("no stream")
    for args, error in (((1, 0, "x", 0, 0, 0, 0, 0, 0), AttributeError), ((1, 0.5, 0, 0, 0, 0, 0, 0, 0), TypeError),
                        ((1, 0, 0, 0, 0, 0, 0, 0, object()), AttributeError), ((1, 0), TypeError)):
        with pytest.raises(error):
            m.run(*args)
    m.bind_stream(broken, lambda: 0)
    with pytest.raises(RuntimeError, match="no stream"):
        m.run(1, 0, 0, 0, 0, 0, 0, 0, None)
    assert seen == []
    with tf.Problem(64, 64, 64) as p:
        assert p.run.__self__ is p           # (run is an ordinary method)


class Data:
    def __init__(self, p): self.p = p
    def data_ptr(self): return self.p


class Index:
    def __index__(self): return 3


@pytest.mark.parametrize("three", [3, np.int64(3), np.uint8(3), torch.tensor(3), C.c_int32(3), Index(), True], ids=lambda x: type(x).__name__)
def test_integers_of_any_type_reach_the_library(three):
    """A variant id straight from numpy's argmin, say. The library sees the number: it knows no such variant."""
    with tf.Problem(0, 64, 64) as p:
        n = len(p.variants())
        assert n == 1
        with pytest.raises(tf.TfError, match="variant id %d out of range" % int(getattr(three, "value", three))):
            p.run(three, 16, 16, 16, 16, stream=0)
        with pytest.raises(tf.TfError, match="variant id 7 out of range"):
            p.run(7, Data(16), 16, 16, 16, workspace=16, workspace_bytes=C.c_size_t(3) if isinstance(three, C.c_int32) else three, stream=0)
    for bad in (0.5, "3", None):
        with tf.Problem(0, 64, 64) as p, pytest.raises(C.ArgumentError):
            p.run(bad, 16, 16, 16, 16, stream=0)


def test_no_address_and_no_handle_are_null(call):
    m, seen = call

    class Stream:
        cuda_stream = None
    m.run(1, 0, Data(None), 0, 0, 0, 0, 0, Stream())
    assert seen == [(1, 0) + (None,) * 5 + (0, None)]


def test_the_module_is_this_interpreters_and_not_needed(monkeypatch, tmp_path):
    """Its file name carries the interpreter's tag, so that another one does not load it; without it (or without what it is
    built with) the library loads, and Problem.run reaches it all the same."""
    assert os.path.basename(tf.PYCALL_PATH) == "_tfcall" + sysconfig.get_config_var("EXT_SUFFIX") == os.path.basename(build.PYCALL)
    assert tf._pycall.__file__ == tf.PYCALL_PATH
    monkeypatch.setattr(tf, "_lib", None)
    monkeypatch.setattr(tf, "_pycall", None)
    monkeypatch.setattr(tf, "_run", None)
    monkeypatch.setattr(tf, "PYCALL_PATH", str(tmp_path / "missing.so"))
    with tf.Problem(0, 64, 64) as p, pytest.raises(tf.TfError, match="variant id 7 out of range"):
        assert tf._pycall is None
        p.run(7, Data(16), 16, 16, 16, stream=0)
    monkeypatch.setattr(build, "PYCALL", str(tmp_path / "_tfcall.so"))
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_pycall() is None and not os.listdir(tmp_path)


def test_a_forked_child_asks_torch_again(call):
    m, seen = call
    m.bind_stream(lambda dev: 100 + dev, lambda: 2)
    pid = os.fork()
    if pid == 0:
        ok = False
        try:
            m.run(1, 0, 0, 0, 0, 0, 0, 0, None)
            ok = seen[-1][-1] == 77              # torch.cuda's own way, which refuses a forked child
        finally:
            os._exit(0 if ok else 1)
    assert os.waitpid(pid, 0)[1] == 0
    m.run(1, 0, 0, 0, 0, 0, 0, 0, None)
    assert [s[-1] for s in seen] == [102]


def test_calls_from_several_threads(call):
    m, seen = call
    here = threading.local()
    m.bind_stream(lambda dev: 1000 * here.n, lambda: 0)

    def work(n):
        here.n = n
        for i in range(200):
            m.run(n, i, n, 2 * n, 3 * n, 4 * n, 0, i, None)
    ts = [threading.Thread(target=work, args=(n,)) for n in range(1, 5)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert sorted(seen) == [(n, i, n, 2 * n, 3 * n, 4 * n, None, i, 1000 * n) for n in range(1, 5) for i in range(200)]


@pytest.mark.gpu
def test_the_current_stream_of_the_calling_thread(call):
    """Without a stream argument the call goes to torch's current stream: of this thread, and of another."""
    m, seen = call
    cb = RUN(lambda *a: seen.append(a) or 0)
    m.bind(C.cast(cb, C.c_void_p).value, tf._current_stream)
    torch.zeros(1, device="cuda")
    got = []

    def work(s):
        with torch.cuda.stream(s):
            for _ in range(2):                   # the slow way once, then torch's C functions
                m.run(1, 0, 0, 0, 0, 0, 0, 0, None)
                got.append((seen[-1][-1] or 0, s.cuda_stream))
    for s in (torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()):
        work(s)
        t = threading.Thread(target=work, args=(s,))
        t.start()
        t.join()
    assert len(got) == 12 and all(a == b for a, b in got)
