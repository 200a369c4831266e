"""The native route's dealings with the interpreter (csrc/calls.cpp), on the CPU: entry points that throw, threads that outlive the interpreter."""
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
