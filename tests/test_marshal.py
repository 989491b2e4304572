"""The native argument marshalling (module _marshal) against the general way
in Python: with the library's entry points replaced by recorders, both make
the same call with the same arguments, over every form of argument that the
native way takes; what it does not take it refuses without a call, and the
binding then converts or rejects it as it always did.  (Device tensors need
the GPU; the refusals of host tensors run on the CPU.)"""
import ctypes

import numpy as np
import pytest

import paper_1601_04033_amd as fa

P = 1000
i32, i64, f32, u64, sz, ptr = (ctypes.c_int32, ctypes.c_int64, ctypes.c_float, ctypes.c_uint64, ctypes.c_size_t,
                               ctypes.c_void_p)
S = "state"
# argument kinds of the C ABI: a ctypes type, or ("array", type, index of its length's argument)
SIGNATURES = {
    "fasgd_apply_updates": [S, ("array", ptr, 4), ("array", i32, 4), ("array", i64, 4), i32, ptr],
    "sasgd_apply_updates": [S, ("array", ptr, 4), ("array", i32, 4), ("array", i64, 4), i32, ptr],
    "bfasgd_select_compact": [S, ptr, f32, f32, u64, i64, i32, ptr, ptr, i64, ptr, ptr, ptr, sz, ptr],
    "bfasgd_select_compact_batch": [S, i32, ("array", ptr, 1), f32, f32, u64, ("array", i64, 1), ("array", i32, 1), ptr,
                                    ptr, i64, ptr, ptr, ptr, sz, ptr],
    "bfasgd_apply_sparse": [S, ptr, ptr, ptr, i64, i32, i64, ptr],
    "fasgd_apply_with_push": [S, ptr, ptr, ptr, ptr, i64, i32, i64, ("array", ptr, 11), ("array", i32, 11),
                              ("array", i64, 11), i32, ptr],
    "fasgd_apply_with_push_and_select": [S, ptr, ptr, ptr, ptr, i64, i32, i64, ("array", ptr, 11), ("array", i32, 11),
                                         ("array", i64, 11), i32, ptr, i32, f32, f32, u64, ptr, ptr, i64, ptr, ptr, ptr,
                                         sz, ptr],
    "fasgd_apply_pushes": [S, i32, ptr, ptr, ptr, ptr, i64, ("array", i32, 1), ("array", i64, 1), ptr],
    "bfasgd_apply_cached": [S, ptr, ptr, ptr, ptr, i64, ptr, i32, i64, ptr],
    "bfasgd_apply_fetch": [ptr, i64, ptr, ptr, ptr, ptr, i64, ptr],
    "bfasgd_decide_segments": [S, ("array", i64, 2, 1), i32, f32, f32, u64, i64, i32, ptr, ptr, sz, ptr],
    "bfasgd_apply_segments": [S, ptr, ("array", i64, 3, 1), i32, ptr, i32, i64, ptr],
}


class Recorder:
    """A stand-in for the loaded library: every entry point records its arguments and returns `status`."""

    def __init__(self):
        self.calls, self.status, self._keep = [], 0, []
        for name, kinds in SIGNATURES.items():
            types = [k if not isinstance(k, (str, tuple)) else ptr for k in kinds]
            setattr(self, name, ctypes.CFUNCTYPE(ctypes.c_int, *types)(self._record(name, kinds)))
        lib = fa.load_library()
        self.bfasgd_list_index_length = lib.bfasgd_list_index_length

    def _record(self, name, kinds):
        def f(*args):
            seen = [name]
            for k, x in zip(kinds, args):
                if isinstance(k, tuple):
                    n = args[k[2]] + (k[3] if len(k) > 3 else 0)
                    seen.append(list(ctypes.cast(x, ctypes.POINTER(k[1]))[:n]))
                else:
                    seen.append(x)
            self.calls.append(seen)
            return self.status
        return f

    def fasgd_last_error(self):
        return b"recorded"


@pytest.fixture
def recorder(monkeypatch):
    native = fa._native()
    rec = Recorder()
    native.bind([ctypes.cast(getattr(rec, n), ptr).value for n in native.ENTRY_POINTS], fa._current_stream)
    monkeypatch.setattr(fa, "load_library", lambda path=None: rec)
    yield rec
    monkeypatch.undo()
    lib = fa.load_library()
    native.bind([ctypes.cast(getattr(lib, n), ptr).value for n in native.ENTRY_POINTS], fa._current_stream)


def test_every_marshalled_entry_point_is_declared():
    assert set(fa._native().ENTRY_POINTS) == set(SIGNATURES) <= set(fa.ABI_FUNCTIONS)


def things(dev):
    import torch
    t = {}
    t["g"] = [torch.zeros(P, device=dev) for _ in range(64)]
    t["idx"] = torch.zeros(P, device=dev, dtype=torch.int32)
    t["val"] = torch.zeros(P, device=dev)
    t["cnt"] = torch.zeros(1, device=dev, dtype=torch.int64)
    t["seg"] = torch.zeros(5 + 3, device=dev, dtype=torch.int32)          # longer than needed: taken
    t["ws"] = torch.zeros(4096, device=dev, dtype=torch.uint8)
    t["bidx"] = torch.zeros(3, 70, device=dev, dtype=torch.int32)
    t["bval"] = torch.zeros(3, 70, device=dev)
    t["bcnt"] = torch.zeros(3, device=dev, dtype=torch.int64)
    t["bseg"] = torch.zeros(3, 5, device=dev, dtype=torch.int32)
    t["send"] = torch.zeros(2, device=dev, dtype=torch.uint8)
    c = fa.fasgd_state()
    c.P, c.lambda_, c.T = P, 8, 100
    t["st"] = fa.State(c, {})
    t["off"] = np.array([0, 400, P], dtype=np.int64)
    return t


def forms(t):
    """(name, arguments, keywords) of calls in every plain form."""
    st, g, idx, val, cnt, seg, ws = (t[k] for k in ("st", "g", "idx", "val", "cnt", "seg", "ws"))
    out = []
    for name in ("fasgd_apply_updates", "sasgd_apply_updates"):
        for K in (1, 2, 31, 64):
            out.append((name, (st, g[:K], [k % 8 for k in range(K)], [90 + k for k in range(K)]), {}))
        out.append((name, (st, tuple(g[:2]), np.array([1, 2], np.int32), (3, np.int64(4))), {}))
    for s in (None, seg):
        out.append(("bfasgd_select_compact", (st, g[0], 5, 1e-8, 2 ** 63 + 5, 7, 3, idx, val, cnt, ws), {"seg_start": s}))
        out.append(("bfasgd_apply_cached", (st, idx, val, cnt, g[2], 2, 9), {"seg_start": s}))
        out.append(("bfasgd_apply_fetch", (g[0], idx, val, cnt), {"seg_start": s}))
        out.append(("fasgd_apply_with_push_and_select",
                    (st, idx, val, cnt, seg, 1, 2, g[:5], [0] * 5, range(5), g[6], 3, 2.5, 0.0, -1, idx, val, cnt, s, ws), {}))
    for s in (None, t["bseg"]):
        out.append(("bfasgd_select_compact_batch", (st, g[:3], 2.5, 0.25, 1, [5, 6, 7], [0, 1, 2], t["bidx"], t["bval"],
                                                    t["bcnt"], ws), {"seg_start": s}))
    out.append(("bfasgd_apply_sparse", (st, idx, val, cnt, np.int32(3), 50), {}))
    out.append(("fasgd_apply_with_push", (st, idx, val, cnt, seg, 1, 2, g[:3], [0, 1, 2], [4, 5, 6]), {}))
    out.append(("fasgd_apply_pushes", (st, t["bidx"], t["bval"], t["bcnt"], t["bseg"], [0, 1, 2], [4, 5, 6]), {}))
    out.append(("bfasgd_decide_segments", (st, t["off"], 1.0, 1e-8, 3, 4, 5, t["send"], ws), {}))
    out.append(("bfasgd_apply_segments", (st, g[0], t["off"], t["send"], 5, 6), {}))
    return out


def general(monkeypatch):
    """The binding's general way alone."""
    class Refuse:
        def __getattr__(self, name):
            return lambda *a: None
    monkeypatch.setattr(fa, "_calls", Refuse())


@pytest.mark.gpu
def test_native_and_general_calls_are_the_same(recorder, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    t = things(torch.device("cuda:0"))
    side = torch.cuda.Stream()
    taken = []

    class Counting:
        def __getattr__(self, name):
            f = getattr(native, name)

            def call(*a):
                rc = f(*a)
                taken.append((name, rc))
                return rc
            return call
    native = fa._native()
    calls = forms(t)
    calls += [(n, a, dict(kw, stream=side)) for n, a, kw in calls]
    calls += [("bfasgd_apply_sparse", (t["st"], t["idx"], torch.nn.Parameter(t["val"]), t["cnt"], 3, 50), {})]
    for name, args, kw in calls:
        with monkeypatch.context() as m:
            m.setattr(fa, "_calls", Counting())
            getattr(fa, name)(*args, **kw)
        with monkeypatch.context() as m:
            general(m)
            getattr(fa, name)(*args, **kw)
        assert taken and taken.pop() == (name, 0), name
        assert len(recorder.calls) == 2 and recorder.calls[0] == recorder.calls[1], (name, kw, recorder.calls)
        recorder.calls.clear()
    with torch.cuda.stream(side):        # the current stream is looked up at each call
        fa.bfasgd_apply_sparse(t["st"], t["idx"], t["val"], t["cnt"], 3, 50)
    assert recorder.calls.pop()[-1] == side.cuda_stream
    recorder.status = 2                  # the library's errors come through
    with pytest.raises(fa.FasgdError, match="recorded"):
        fa.bfasgd_apply_sparse(t["st"], t["idx"], t["val"], t["cnt"], 3, 50)


def refusals(t, torch):
    """(arguments of fasgd_apply_updates / bfasgd_apply_sparse / ..., the exception of the general way or None)."""
    st, g, idx, val, cnt = t["st"], t["g"], t["idx"], t["val"], t["cnt"]

    class Mine(torch.Tensor):
        pass

    mine = val.clone().as_subclass(Mine)
    return [
        ("fasgd_apply_updates", (st, [], [], []), ValueError),
        ("fasgd_apply_updates", (st, g[:1] * 65, [0] * 65, [0] * 65), ValueError),
        ("fasgd_apply_updates", (st, g[:2], [0], [0, 0]), ValueError),
        ("fasgd_apply_updates", (st, g[:2], [0, 0], [0]), ValueError),
        ("fasgd_apply_updates", (st, [g[0][:-1]], [0], [0]), ValueError),
        ("fasgd_apply_updates", (st, [g[0].double()], [0], [0]), TypeError),
        ("fasgd_apply_updates", (st, [None], [0], [0]), AttributeError),
        ("fasgd_apply_updates", (st, g[:1], ["x"], [0]), ValueError),
        ("bfasgd_apply_sparse", (st, idx, val[:-1], cnt, 0, 0), ValueError),
        ("bfasgd_apply_sparse", (st, idx.long(), val, cnt, 0, 0), TypeError),
        ("bfasgd_apply_sparse", (st, idx, val, cnt.int(), 0, 0), TypeError),
        ("bfasgd_apply_sparse", (st, idx, torch.zeros(2 * P, device=val.device)[::2], cnt, 0, 0), TypeError),
        ("bfasgd_apply_sparse", (st, idx, mine, cnt, 0, 0), None),
        ("bfasgd_apply_sparse", (st, idx, val, cnt, 1.0, 2.5), None),
        ("fasgd_apply_pushes", (st, t["bidx"], t["bval"][:2], t["bcnt"], t["bseg"], [0, 1, 2], [0, 0, 0]), ValueError),
        ("fasgd_apply_pushes", (st, t["bidx"], t["bval"], t["bcnt"], t["bseg"][:, :4], [0, 1, 2], [0, 0, 0]), ValueError),
        ("fasgd_apply_with_push", (st, idx, val, cnt, None, 1, 2, g[:1], [0], [0]), ValueError),
        ("fasgd_apply_with_push", (st, idx, val, cnt, t["seg"][:4], 1, 2, g[:1], [0], [0]), ValueError),
        ("bfasgd_apply_segments", (st, g[0], [0, 400, P], t["send"], 5, 6), None),
        ("bfasgd_apply_segments", (st, g[0], t["off"].astype(np.int32), t["send"], 5, 6), None),
        ("bfasgd_decide_segments", (st, t["off"], 1.0, 1e-8, 3, 4, 5, t["send"][:1], t["ws"]), ValueError),
    ]


@pytest.mark.gpu
def test_what_is_not_plain_goes_the_general_way(recorder):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    t = things(torch.device("cuda:0"))
    native = fa._native()
    native_args = {"bfasgd_apply_sparse": lambda a: (a[0].c, *a[1:], None),
                   "fasgd_apply_updates": lambda a: (a[0].c, *a[1:], None),
                   "fasgd_apply_pushes": lambda a: (a[0].c, *a[1:], None),
                   "fasgd_apply_with_push": lambda a: (a[0].c, *a[1:], None),
                   "bfasgd_apply_segments": lambda a: (a[0].c, *a[1:], None),
                   "bfasgd_decide_segments": lambda a: (a[0].c, *a[1:], None)}
    for name, args, error in refusals(t, torch):
        assert getattr(native, name)(*native_args[name](args)) is None, (name, args)
        assert not recorder.calls, name
        if error is None:
            getattr(fa, name)(*args)
            assert len(recorder.calls) == 1, name
            recorder.calls.clear()
        else:
            with pytest.raises(error):
                getattr(fa, name)(*args)
            assert not recorder.calls, name


def test_host_tensors_are_refused(recorder):
    """Host tensors reach neither the library nor the current stream; the general way rejects them by name."""
    import torch
    t = things(torch.device("cpu"))
    for name, args, kw in forms(t):
        with pytest.raises(TypeError, match="must be a CUDA"):
            getattr(fa, name)(*args, **kw)
    assert not recorder.calls


def test_wrong_arity_and_binding_are_errors():
    native = fa._native()
    with pytest.raises(TypeError):
        native.fasgd_apply_updates(1, 2)
    with pytest.raises(ValueError):
        native.bind([0] * len(SIGNATURES), fa._current_stream)
    with pytest.raises(ValueError):
        native.bind([1], fa._current_stream)


class Raises:
    """A number whose conversion raises."""

    def __init__(self, e):
        self.e = e

    def __index__(self):
        raise self.e

    __int__ = __index__


@pytest.mark.parametrize("e", [KeyboardInterrupt, MemoryError, RuntimeError, SystemExit])
def test_exceptions_that_are_no_refusal_come_out(recorder, e):
    """What a signal handler (or the interpreter) raises while a number is converted ends the call."""
    import torch
    t = things(torch.device("cpu"))
    st, off = t["st"], t["off"]
    native = fa._native()
    with pytest.raises(e):
        native.bfasgd_decide_segments(st.c, off, 1.0, 1e-8, 3, Raises(e()), 5, t["send"], t["ws"], None)
    with pytest.raises(e):
        native.fasgd_apply_pushes(st.c, t["bidx"], t["bval"], t["bcnt"], t["bseg"], [0, Raises(e()), 2], [0, 0, 0], None)
    with pytest.raises(e):
        native.fasgd_apply_pushes(st.c, t["bidx"], t["bval"], t["bcnt"], t["bseg"], [0, 1, 2], [0, 0, Raises(e())], None)
    # those that say "not plain" are the general way's to raise
    for mild in (TypeError(), ValueError(), OverflowError()):
        assert native.bfasgd_decide_segments(st.c, off, 1.0, 1e-8, 3, Raises(mild), 5, t["send"], t["ws"], None) is None
    assert not recorder.calls


@pytest.mark.gpu
@pytest.mark.parametrize("e", [KeyboardInterrupt, TypeError])
def test_the_stream_lookup_s_exception_comes_out(recorder, e):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    t = things(torch.device("cuda:0"))
    native = fa._native()

    def lookup():
        raise e()
    native.bind([ctypes.cast(getattr(recorder, n), ptr).value for n in native.ENTRY_POINTS], lookup)
    with pytest.raises(e):                       # the recorder's fixture binds the library again
        fa.bfasgd_apply_sparse(t["st"], t["idx"], t["val"], t["cnt"], 3, 50)
    assert not recorder.calls


def test_a_list_that_shrinks_while_it_is_read(recorder):
    """A number whose conversion shortens its own list: the list's new length is seen, and the call is refused."""
    import torch
    t = things(torch.device("cpu"))
    seen = []

    class Shrinks:
        def __index__(self):
            del clients[1:]
            return 1

    class Seen:
        def __index__(self):
            seen.append(1)
            return 2
    clients = [Shrinks(), 1, 2]
    assert fa._native().fasgd_apply_pushes(t["st"].c, t["bidx"], t["bval"], t["bcnt"], t["bseg"], clients, [Seen(), 1, 1],
                                           None) is None
    assert len(clients) == 1 and not seen and not recorder.calls


def test_a_short_transmit_array_is_rejected(recorder):
    """The segment apply reads one byte per segment: an array made for fewer segments does not reach the library."""
    import torch
    t = things(torch.device("cpu"))
    with pytest.raises(ValueError, match="one entry per segment"):
        fa.bfasgd_apply_segments(t["st"], t["g"][0], t["off"], t["send"][:1], 5, 6)
    assert not recorder.calls


@pytest.mark.gpu
def test_transmit_arrays_on_the_device(recorder):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    t = things(torch.device("cuda:0"))
    for off in (t["off"], t["off"].tolist()):    # the native and the general way
        with pytest.raises(ValueError, match="one entry per segment"):
            fa.bfasgd_apply_segments(t["st"], t["g"][0], off, t["send"][:1], 5, 6)
        assert not recorder.calls
        fa.bfasgd_apply_segments(t["st"], t["g"][0], off, torch.zeros(3, device="cuda:0", dtype=torch.uint8), 5, 6)
        assert len(recorder.calls) == 1          # a longer array is taken
        recorder.calls.clear()


@pytest.fixture
def unbound(recorder, monkeypatch):
    """The binding before its first call, on a recorder, with host tensors taken for device ones."""
    monkeypatch.setattr(fa, "_calls", None)
    monkeypatch.setattr(fa, "_dev_ptr", lambda t, *a: None if t is None else t.data_ptr())
    monkeypatch.setattr(fa, "_stream", lambda stream: 0)
    yield recorder


def _every_call_is_served(recorder):
    import torch
    t = things(torch.device("cpu"))
    with pytest.warns(RuntimeWarning, match="marshalled in Python") as seen:
        for name, args, kw in forms(t):
            getattr(fa, name)(*args, **kw)
            assert recorder.calls.pop()[0] == name and not recorder.calls
    assert len(seen) == 1


def test_without_the_module_calls_are_marshalled_in_python(unbound, monkeypatch):
    import sys
    monkeypatch.delattr(fa, "_marshal", raising=False)
    monkeypatch.setitem(sys.modules, fa.__name__ + "._marshal", None)     # its import fails
    _every_call_is_served(unbound)


def test_a_module_of_another_torch_is_not_used(unbound, monkeypatch):
    import torch
    monkeypatch.setattr(torch, "__version__", "0.1")
    _every_call_is_served(unbound)


def test_the_library_is_built_without_a_host_compiler(tmp_path, monkeypatch, capsys):
    import paper_1601_04033_amd._build as lib_build
    old = tmp_path / "_marshal.so"
    old.write_bytes(b"")
    monkeypatch.setattr(lib_build, "MARSHAL", str(old))
    monkeypatch.setenv("CXX", "no-such-compiler")
    assert lib_build.build_marshal() is None
    assert "left out" in capsys.readouterr().err and not old.exists()


@pytest.mark.parametrize("c,eps_c,seed", [(np.float64(1.0), np.float32(1e-8), np.int64(3)), (np.int32(1), 0, np.uint64(2 ** 63)),
                                          (True, 1e-8, False)])
def test_numpy_numbers_are_plain(recorder, c, eps_c, seed):
    """Numbers that ctypes and int() convert are not left to the general way: the timestamp after them is reached."""
    import torch
    t = things(torch.device("cpu"))
    with pytest.raises(KeyboardInterrupt):
        fa._native().bfasgd_decide_segments(t["st"].c, t["off"], c, eps_c, seed, Raises(KeyboardInterrupt()), 5, t["send"],
                                            t["ws"], None)


@pytest.mark.gpu
def test_raw_streams_and_numpy_numbers_are_marshalled_natively(recorder, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    t = things(torch.device("cuda:0"))
    st, g, idx, val, cnt, ws = (t[k] for k in ("st", "g", "idx", "val", "cnt", "ws"))
    side = torch.cuda.Stream()
    for s in (0, int(side.cuda_stream), side, None):
        for args in ((st, g[0], np.float64(2.5), np.float32(1e-8), np.uint64(2 ** 64 - 1), 7, 3, idx, val, cnt, ws),
                     (st, g[0], 0.1, 0, np.int64(-5), np.int64(7), np.int32(3), idx, val, cnt, ws)):
            assert fa._native().bfasgd_select_compact(st.c, *args[1:], None, s) == 0
            with monkeypatch.context() as m:
                general(m)
                fa.bfasgd_select_compact(*args, stream=s)
            assert len(recorder.calls) == 2 and recorder.calls[0] == recorder.calls[1], (s, recorder.calls)
            recorder.calls.clear()
