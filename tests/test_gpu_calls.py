"""The native route from Python arguments to the entry points (csrc/calls.cpp) against the ctypes route: the same values reach the library, and what is
not of the plain form is left to the latter.  The entry points are stand-ins that note what they are given; nothing is launched."""
import ctypes

import pytest
import torch

from paper_2411_01109_amd import binding

H, F32 = torch.float16, torch.float32


def arguments(dev):
    """entry -> (positional arguments, keyword arguments) of calls; every tensor, size and number is another one."""
    def table(n, f, pad=8, dtype=H):
        return torch.empty((n, f + pad), dtype=dtype, device=dev)[:, :f]

    def edge(n, dtype=H):
        return torch.empty((n, 2), dtype=dtype, device=dev)

    ints = lambda n: torch.zeros(n, dtype=torch.int32, device=dev)  # noqa: E731
    g, gt = binding.Csr(ints(6), ints(9), ncols=7), binding.Csr(ints(8), ints(9), ncols=5, eid=ints(9))
    p, pt = binding.Plan(0x7f0010, g), binding.Plan(0x7f0020, gt)
    ws = torch.empty(77, dtype=torch.int32, device=dev)
    X, Y, Z, W = table(5, 16), table(5, 24, 16), table(7, 40), table(16, 24, 0)
    v16, v32 = torch.empty(16, dtype=H, device=dev), torch.empty(24, dtype=F32, device=dev)
    param = torch.nn.Parameter(table(16, 24, 0))
    return g, gt, p, pt, {
        "hgnn_linear": [((X, W, Y), {}), ((X, param, Y), {}), ((X, table(24, 16), Y), {"trans_w": True}), ((table(5, 32), W, Y), {"K": 24, "F": 20}),
                        ((X, W, Y), {"stream": 0x1230})],
        "hgnn_linear_wgrad": [((X, Y, table(16, 24, 4, F32), ws), {}), ((X, Y, table(16, 24, 4, F32), ws), {"K": 8, "F": 16})],
        "hgnn_spmm": [((g, None, 1, Z, Y), {}), ((g, edge(9), 2, Z, Y), {"op": 1, "row_scale": v32, "F": 12, "workspace": ws})],
        "hgnn_spmm_discretized": [((p, g, None, 1, Z, Y), {}), ((p, gt, edge(9), 2, Z, Y), {"op": 1, "row_scale": v32, "F": 12, "stream": 0})],
        "hgnn_spmm_discretized_fused": [((p, g, None, 1, Z, Y), {}),
                                        ((p, g, edge(9), 2, Z, Y), dict(op=1, row_scale=v32, col_scale=v32[3:], self_feat=X, self_coef=1.25, agg_coef=0.1,
                                                                        F=10, scaled_x=table(7, 48)))],
        "hgnn_sddmm": [((g, None, 0, 1, 16, X, Z, edge(9)), {}), ((g, p, 1, 2, 8, X, Z, edge(9), v16, v16[8:], 0.3), {})],
        "hgnn_edge_softmax": [((g, None, 2, edge(9), edge(9)), {}), ((g, p, 2, edge(9), edge(9)), {"stream": 5})],
        "hgnn_edge_softmax_bwd": [((g, p, 2, edge(9), edge(9), edge(9)), {}), ((g, None, 2, edge(9), edge(9), edge(9)), {"e": edge(9), "neg_slope": 0.4})],
        "hgnn_edge_rowsum": [((gt, pt, 2, edge(9), edge(7)), {}), ((gt, None, 2, edge(9), edge(7)), {})],
        "hgnn_edge_colsum": [((g, p, 1, edge(9), edge(7)), {})],
        "hgnn_gat_forward_fused": [((g, p, 2, 8, X, Z, v16, v16[8:], Y), {}), ((g, p, 2, 8, X, Z, v16, v16[8:], Y, v32), {"neg_slope": 0.1})],
        "hgnn_gat_forward_fused_save": [((g, p, 2, 8, X, Z, v16, v16[8:], Y, v32, table(5, 8), v32[2:]), {"neg_slope": 0.1})],
        "hgnn_gat_backward_fused_saved": [((g, p, gt, pt, 2, 8, X, Z, v16, v16[8:], Y, v32, table(5, 8), v32[2:], table(5, 56), table(7, 64), v16[1:], v16[2:]),
                                           {"neg_slope": 0.1})],
        "hgnn_gat_feature_grad": [((2, 8, X, v16, v16[2:], v16[4:], v16[6:], Y, Z, v32, v32[5:], ws), {})],
    }


def plain(v):
    """an argument as it reaches the library"""
    if v is None:
        return 0
    if hasattr(v, "_obj"):  # byref
        s = v._obj
        return tuple(plain(getattr(s, f)) for f, _ in s._fields_)
    if hasattr(v, "contents"):
        return tuple(plain(getattr(v.contents, f)) for f, _ in v.contents._fields_)
    return ctypes.c_float(v).value if isinstance(v, float) else int(v)


class StandIn:
    def __init__(self, lib, seen):
        self.lib, self.seen = lib, seen

    def __getattr__(self, name):
        if not name.startswith("hgnn_") or name in ("hgnn_status_str", "hgnn_last_error"):
            return getattr(self.lib, name)
        return lambda *a: self.seen.append((name, tuple(plain(v) for v in a))) or 0


@pytest.fixture
def routes(hgnn, monkeypatch):
    """-> (native module bound to stand-ins, what they have seen); bound to the library again afterwards"""
    lib, native, seen = hgnn.load(), binding._calls, []
    assert native is not None
    keep, addresses = [], {}
    for name in hgnn.EXPORTS:
        fn = getattr(lib, name)
        if fn.argtypes and fn.restype in (None, ctypes.c_int):
            kind = ctypes.CFUNCTYPE(ctypes.c_int, *fn.argtypes)
            keep.append(kind(lambda *a, name=name: seen.append((name, tuple(plain(v) for v in a))) or 0))
            addresses[name] = ctypes.cast(keep[-1], ctypes.c_void_p).value
    native.bind(addresses, binding._raw_stream, binding._current_device)
    monkeypatch.setattr(binding, "load", lambda: StandIn(lib, seen))
    yield native, seen
    native.bind({n: ctypes.cast(getattr(lib, n), ctypes.c_void_p).value for n in hgnn.EXPORTS}, binding._raw_stream, binding._current_device)


@pytest.mark.gpu
def test_the_same_arguments_arrive(hgnn, dev, routes, monkeypatch):
    native, seen = routes
    g, gt, p, pt, calls = arguments(dev)
    streams = [None, torch.cuda.Stream()]
    for name, forms in calls.items():
        for args, kw in forms:
            for s in streams:
                with torch.cuda.stream(s or torch.cuda.current_stream()):
                    del seen[:]
                    assert getattr(native, name[5:]) is not None
                    monkeypatch.setattr(binding, "_calls", native)
                    getattr(hgnn, name)(*args, **kw)
                    monkeypatch.setattr(binding, "_calls", None)
                    getattr(hgnn, name)(*args, **kw)
                assert len(seen) == 2 and seen[0] == seen[1], (name, kw, seen)
    p.handle = pt.handle = None  # (not the library's)


@pytest.mark.gpu
def test_other_forms_are_left_alone(hgnn, dev, routes, monkeypatch):
    native, seen = routes
    g, gt, p, pt, calls = arguments(dev)
    X, W, Y = calls["hgnn_linear"][0][0]

    class Sub(torch.Tensor):
        pass

    stream = torch.cuda.Stream()
    taken = [((X, W, Y, 1), {}), ((X.as_subclass(Sub), W, Y), {}), ((X, W, Y), {"stream": stream}), ((X, W, Y), {"K": True})]
    for args, kw in taken:  # by the ctypes route, with the same values as ever
        del seen[:]
        hgnn.hgnn_linear(*args, **kw)
        assert len(seen) == 1, (args, kw)
    refused = [((X.float(), W, Y), TypeError), ((X, W.cpu(), Y), TypeError), ((X, W, Y.t()), ValueError), ((X[0], W, Y), IndexError),
               ((X, W, None), AttributeError), ((X, W, "Y"), AttributeError)]
    for args, error in refused:
        got = []
        for route in (native, None):
            monkeypatch.setattr(binding, "_calls", route)
            del seen[:]
            with pytest.raises(error) as e:
                hgnn.hgnn_linear(*args)
            got.append(str(e.value))
            assert not seen
        assert got[0] == got[1]
    p.handle = pt.handle = None


def test_nothing_is_called_for_what_is_not_plain(hgnn):
    """On the CPU no argument is a GPU tensor: every function hands the call back, whatever it is given."""
    hgnn.load()
    calls = binding._calls
    if calls is None:
        pytest.skip("torch without a current raw stream")
    t = torch.zeros((4, 8), dtype=H)
    for n in range(24):
        for v in (t, None, 1, "x", 1.0, object()):
            for name in ("linear", "linear_wgrad", "spmm", "spmm_discretized", "spmm_discretized_fused", "sddmm", "edge_softmax", "edge_softmax_bwd",
                         "edge_rowsum", "edge_colsum", "gat_forward_fused", "gat_forward_fused_save", "gat_backward_fused_saved", "gat_feature_grad"):
                assert getattr(calls, name)(*([v] * n)) == -1
    with pytest.raises(TypeError):
        calls.bind(1)
    with pytest.raises(KeyError):
        calls.bind({}, None, None)


def test_no_thread_local_memory():
    """A library with thread-local memory that is loaded late and does not use it slows every access to such memory in the runtime down (glibc's slow
    way for modules older than the newest one): set-up calls took 2 us more."""
    with open(binding.CALLS_PATH, "rb") as fh:
        head = fh.read(64)
        assert head[:5] == b"\x7fELF\x02"
        at, size, n = int.from_bytes(head[32:40], "little"), int.from_bytes(head[54:56], "little"), int.from_bytes(head[56:58], "little")
        fh.seek(at)
        kinds = [int.from_bytes(fh.read(size)[:4], "little") for _ in range(n)]
    assert 1 in kinds and 7 not in kinds  # PT_LOAD, PT_TLS


@pytest.fixture
def taken(hgnn, monkeypatch):
    """-> the list of calls as (route, entry, values), the stand-ins of either route noting theirs"""
    lib, native, log = hgnn.load(), binding._calls, []
    assert native is not None
    keep, addresses = [], {}
    for name in hgnn.EXPORTS:
        fn = getattr(lib, name)
        if fn.argtypes and fn.restype in (None, ctypes.c_int):
            kind = ctypes.CFUNCTYPE(ctypes.c_int, *fn.argtypes)
            keep.append(kind(lambda *a, name=name: log.append(("native", name, tuple(plain(v) for v in a))) or 0))
            addresses[name] = ctypes.cast(keep[-1], ctypes.c_void_p).value

    class Ctypes(StandIn):
        def __getattr__(self, name):
            if not name.startswith("hgnn_") or name in ("hgnn_status_str", "hgnn_last_error"):
                return getattr(self.lib, name)
            return lambda *a: log.append(("ctypes", name, tuple(plain(v) for v in a))) or 0

    native.bind(addresses, binding._raw_stream, binding._current_device)
    monkeypatch.setattr(binding, "load", lambda: Ctypes(lib, log))
    yield log
    native.bind({n: ctypes.cast(getattr(lib, n), ctypes.c_void_p).value for n in hgnn.EXPORTS}, binding._raw_stream, binding._current_device)


def both_ways(hgnn, log, monkeypatch, name, args, kw):
    """-> (route, values) of a call with the native module, after the same without it, whose values must be the same"""
    native = binding._calls
    got = []
    for module in (native, None):
        del log[:]
        monkeypatch.setattr(binding, "_calls", module)
        getattr(hgnn, name)(*args, **kw)
        assert len(log) == 1, (name, kw, log)
        got += log
    monkeypatch.setattr(binding, "_calls", native)
    assert got[1][0] == "ctypes" and got[0][1:] == got[1][1:], (name, kw, got)
    return got[0][0]


@pytest.mark.gpu
def test_plain_calls_are_made_natively(hgnn, dev, taken, monkeypatch):
    g, gt, p, pt, calls = arguments(dev)
    for name, forms in calls.items():
        for args, kw in forms:
            assert both_ways(hgnn, taken, monkeypatch, name, args, kw) == "native", (name, kw)
    p.handle = pt.handle = None  # (not the library's)


@pytest.mark.gpu
def test_streams_and_whole_numbers_are_plain(hgnn, dev, taken, monkeypatch):
    """A stream object, as torch hands it out, and an int where a float is meant cost no second way."""
    g, gt, p, pt, calls = arguments(dev)
    stream = torch.cuda.Stream()

    class Holder:
        cuda_stream = 0x4560

    for name, forms in calls.items():
        args, kw = forms[-1]
        for s in (stream, torch.cuda.current_stream(), torch.cuda.ExternalStream(stream.cuda_stream), Holder(), 0, 0x7f0000001230):
            assert both_ways(hgnn, taken, monkeypatch, name, args, dict(kw, stream=s)) == "native", (name, s)
            assert taken[0][2][-1] == getattr(s, "cuda_stream", s)
        if "neg_slope" in kw:
            assert both_ways(hgnn, taken, monkeypatch, name, args, dict(kw, neg_slope=0)) == "native"
    X, W, Y = calls["hgnn_linear"][0][0]

    class Sub(torch.Tensor):
        pass

    for args, kw in [((X.as_subclass(Sub), W, Y), {}), ((X, W, Y, None), {}), ((X, W, Y), {"stream": "7"}), ((X, W, Y), {"stream": 7.0})]:  # as ever by ctypes
        assert both_ways(hgnn, taken, monkeypatch, "hgnn_linear", args, kw) == "ctypes", (args, kw)
    for args, kw in [((X, W, Y), {"K": True}), ((X, W, Y, 1), {}), ((X, W, Y, 0), {}), ((X, W, Y, 1 << 70), {})]:
        assert both_ways(hgnn, taken, monkeypatch, "hgnn_linear", args, kw) == "native", (args, kw)
    p.handle = pt.handle = None
