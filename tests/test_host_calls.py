"""The native route's dealings with the interpreter (csrc/calls.cpp), on the CPU: entry points that throw, threads that outlive the interpreter;
and the package without the module."""
import os
import subprocess
import sys

import pytest

from paper_2411_01109_amd import build as hip_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    """-> folder with the module calls_probe"""
    d = tmp_path_factory.mktemp("calls")
    hip_build.compile_calls(os.path.join(HERE, "calls_probe.cpp"), str(d / "calls_probe.so"), ["-O1", "-I", hip_build.CSRC])
    return str(d)


def run(folder, text):
    return subprocess.run([sys.executable, "-c", "import sys, threading, time, torch\nsys.path.insert(0, %r)\nfrom calls_probe import probe\n%s" % (folder, text)],
                          capture_output=True, text=True, timeout=120, cwd=os.path.dirname(HERE))


def test_exceptions_of_an_entry_point(probe):
    """They arrive as Python's, with the lock held, and the call does not count as one that has not been made."""
    r = run(probe, """
def one():
    for what, error, text in ((1, MemoryError, ""), (2, RuntimeError, "out of luck")):
        try:
            probe(what)
        except error as e:
            assert str(e) == text, e
        else:
            raise AssertionError(what)
    assert probe(0) == 0 and probe(4) == 1 and probe("x") == -1 and probe(0, 0) == -1
threads = [threading.Thread(target=one) for _ in range(4)]
for t in threads: t.start()
for t in threads: t.join()
one()
print("done")
""")
    assert r.returncode == 0 and r.stdout.endswith("done\n") and not r.stderr, r


def test_a_thread_that_outlives_the_interpreter(probe):
    """A daemon thread inside a call wants the lock back while the interpreter ends, and is unwound: nothing may stop that."""
    r = run(probe, """
class Last:
    def __del__(self, sleep=time.sleep):
        sleep(1.5)
threading.Thread(target=probe, args=(3,), daemon=True).start()
time.sleep(0.1)
sys.modules["__main__"].last = Last()
print("done", flush=True)
""")
    assert r.returncode == 0 and r.stdout == "done\n" and not r.stderr, r


def test_a_graph_that_is_given_another_structure_meanwhile(probe):
    """A call goes on with the graph that it was given, whatever another thread does to the object."""
    r = run(probe, """
from calls_probe import rows_later
from paper_2411_01109_amd.binding import _CsrStruct
class Graph:
    struct = None
g = Graph()
g.struct = _CsrStruct(7, 7, 0, None, None, None, None)
got = []
t = threading.Thread(target=lambda: got.append(rows_later(g)))
t.start()
time.sleep(0.2)
g.struct = None
others = [_CsrStruct(9, 9, 0, None, None, None, None) for _ in range(1000)]
t.join()
assert got == [7], got
print("done")
""")
    assert r.returncode == 0 and r.stdout == "done\n", r


@pytest.mark.parametrize("how", ["missing", "for another interpreter", "there"])
def test_the_library_serves_without_the_module(hgnn, tmp_path, how):
    """The package with the library and without a module of native calls that loads: every call goes through ctypes, as it does for arguments that are not plain."""
    pkg = tmp_path / "paper_2411_01109_amd"
    pkg.mkdir()
    here = os.path.dirname(hip_build.LIB_PATH)
    for name in ("__init__.py", "binding.py", "libhgnn.so", "_calls.so"):
        if name != "_calls.so" or how == "there":
            os.symlink(os.path.join(here, name), str(pkg / name))
    if how == "for another interpreter":
        (pkg / "_calls.so").write_bytes(b"not of this world")
    text = """
import warnings
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    from paper_2411_01109_amd import binding
    lib = binding.load()
    assert binding.load() is lib
assert binding.hgnn_linear_wgrad_workspace(64, 64) > 0
print((binding._calls is not None), [str(x.category.__name__) for x in w if "_calls" in str(x.message)])
try:
    binding.hgnn_linear(torch.zeros(4, 8).half(), torch.zeros(8, 8).half(), torch.zeros(4, 8).half())
except TypeError as e:
    assert "CUDA (HIP)" in str(e)
else:
    raise AssertionError("a tensor on the CPU was taken")
"""
    r = subprocess.run([sys.executable, "-c", "import sys, torch\nsys.path.insert(0, %r)\n%s" % (str(tmp_path), text)], capture_output=True, text=True,
                       timeout=120, cwd=str(tmp_path))
    want = {"missing": "False []", "for another interpreter": "False ['RuntimeWarning']", "there": "True []"}[how]
    assert r.returncode == 0 and r.stdout.strip() == want, r
