"""The binding's native calls: what reaches the C function, and which arguments are left to the Python function."""
import copy
import ctypes
import inspect
import pickle

import pytest

L, I, P, Z, F, INT = ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_float, ctypes.c_int
RUN = [P, L, P, L, I, P, I, P, L]
WS = [P, Z, P]
KINDS = {                                                # the C functions' arguments as include/ngemm.h declares them
    "run": RUN + WS, "static": RUN + [P], "requant": RUN[:7] + [F, I, P, L] + WS,
    "channel": RUN[:7] + [P, P, P, I, I, P, L] + WS, "unpacked": [P, L, L, L, P, L, I, P, L, I, P, L] + WS,
    "batched": [P, INT, P] + WS, "pack": [P, L, L, P, L, P, Z, P, ctypes.POINTER(P)], "free": [P],
}
NAMES = {"run": "ngemm_run_u8s8s32", "static": "ngemm_run_u8s8s32_static", "requant": "ngemm_run_u8s8u8_requant",
         "channel": "ngemm_run_u8s8u8_requant_channel", "unpacked": "ngemm_run_u8s8s32_unpacked",
         "batched": "ngemm_run_batched_u8s8s32", "pack": "ngemm_pack_b", "free": "ngemm_packed_b_free"}


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


class Stream:
    cuda_stream = 0x5eed


def forget_streams():
    """What the binding knows of the current stream: nothing, so that the next call without a stream looks for it."""
    from paper_1910_00178_amd import binding
    binding._calls.streams(None, None, None)
    binding._current_stream = binding._slow_current_stream


def watched_calls():
    """both(kind, status) -> (native call, what the C function saw, what the Python function was given)"""
    from paper_1910_00178_amd import binding
    forget_streams()
    keep = []

    def make(kind, status=0):
        seen, given = [], []

        def c(*a):
            seen.append(a)
            if kind == "pack":
                a[-1][0] = 0x1234
            return status

        def slow(*a, **kw):
            given.append((a, kw))
            return "slow"
        slow.__name__ = NAMES[kind]
        fn = ctypes.CFUNCTYPE(INT, *KINDS[kind])(c)
        keep.append(fn)
        return binding._calls.Call(slow, kind, ctypes.cast(fn, P).value), seen, given
    yield make
    forget_streams()


both = pytest.fixture(watched_calls, name="both")


def usual(kind):
    """Arguments of the usual types for every parameter of the Python function, and what the C function has to see."""
    from paper_1910_00178_amd import binding
    fn = getattr(binding, NAMES[kind])
    problems = binding.make_problems([(1, 2, 3, 4, 5, 6, 7, 8)] * 3)
    args, want = [], []
    for n, name in enumerate(inspect.signature(fn).parameters):
        at = 0x1000 * (n + 1)
        if name in ("ctx", "B", "b"): a, w = P(at), at
        elif name == "problems":
            a, w = problems, ctypes.addressof(problems)
            want.append(3)
        elif name == "hip_stream": a, w = Stream(), 0x5eed
        elif name == "scale": a, w = 0.1, F(0.1).value
        elif name == "relu": a, w = True, 1
        elif name.endswith("_zero_point"): a, w = -3 - n, -3 - n
        elif name.endswith(("_dev",)): a, w = Tensor(at), at
        else: a, w = (1 << 40) + n, (1 << 40) + n
        args.append(a)
        want.append(w)
    return args, want


@pytest.mark.parametrize("kind", KINDS)
def test_native_call(both, kind):
    call, seen, given = both(kind)
    args, want = usual(kind)
    out = call(*args)
    assert not given and len(seen) == 1 and list(seen[0])[:len(want)] == want
    if kind == "pack":
        assert type(out) is P and out.value == 0x1234
    else:
        assert out is None
    # handles as integers, empty pointers
    call(*[a.value if type(a) is P else None if isinstance(a, Tensor) else a for a in args])
    assert not given and list(seen[1])[:len(want)] == [None if isinstance(a, Tensor) else w for a, w in
                                                       zip(args if kind != "batched" else [None] + args, want)]
    # every other way of saying it goes to the Python function untouched, nothing having been called
    others = {P: ("0", 1.5, -1), Tensor: ("0", 1.5, -1, object()), Stream: ("0", 1.5, -1), float: (1, "x"), bool: ("x", None), int: (1.0, "1", 1 << 70, True)}
    for n, a in enumerate(args):
        for other in others.get(type(a), (None, 1, object(), (ctypes.c_int * 3)())):
            bad = args[:n] + [other] + args[n + 1:]
            assert call(*bad) == "slow" and given.pop()[0] == tuple(bad)
    if kind != "free":
        params = list(inspect.signature(call).parameters)
        assert params == list(inspect.signature(call.__wrapped__).parameters)
        assert call(*args[:1], **{"x": 1}) == "slow" and given.pop()[1] == {"x": 1}
    assert call() == "slow" and call(*args, 1) == "slow"
    assert len(seen) == 2


def test_defaults_and_stream(both):
    from paper_1910_00178_amd import binding
    call, seen, given = both("run")
    args, _ = usual("run")
    assert call(*args[:9]) == "slow"                      # the current stream is not known yet: the Python function finds it
    up = [True]
    binding._calls.streams(lambda d: 0x100 + d, lambda: 7, lambda: up[0])
    assert call(*args[:9]) is None and seen[-1][9:] == (None, 0, 0x107)
    assert call(*args[:11], None) is None and seen[-1][11] == 0x107
    assert call(*args[:11], 0) is None and seen[-1][11] is None
    up[0] = False                                         # not initialised, or a forked child
    n = len(seen)
    assert call(*args[:9]) == "slow" and len(seen) == n
    assert len(given) == 2


def test_these_tests_leave_the_stream_to_be_found():
    from paper_1910_00178_amd import binding
    steps = watched_calls()
    next(steps)
    binding._calls.streams(lambda d: 1, lambda: 2, lambda: True)
    binding._current_stream = lambda: 4                   # as a call that has found it leaves them
    next(steps, None)
    assert binding._current_stream is binding._slow_current_stream


def test_whole_numbers_at_their_ends(both):
    call, seen, given = both("run")
    args, _ = usual("run")
    for n, lo, hi in ((1, -2**63, 2**63 - 1), (4, -2**31, 2**31 - 1), (10, 0, 2**63 - 1)):
        for v in (lo, hi):
            call(*args[:n], v, *args[n + 1:])
            assert not given and seen[-1][n] == v
        for v in (lo - 1, hi + 1):
            assert call(*args[:n], v, *args[n + 1:]) == "slow" and given.pop()


def test_errors_and_interrupts(both):
    from paper_1910_00178_amd import binding
    call, _, _ = both("run", status=-2)
    args, _ = usual("run")
    with pytest.raises(binding.NgemmError, match="ngemm_run_u8s8s32: bad shape") as e:
        call(*args)
    assert e.value.status == -2

    class Interrupted:
        def data_ptr(self):
            raise KeyboardInterrupt
    with pytest.raises(KeyboardInterrupt):
        call(*args[:2], Interrupted(), *args[3:])


def test_binding_holds_them():
    import paper_1910_00178_amd as ng
    from paper_1910_00178_amd import binding
    for kind, name in NAMES.items():
        fn = getattr(ng, name)
        assert type(fn) is binding._calls.Call and fn.__name__ == name and inspect.signature(fn) == inspect.signature(fn.__wrapped__)
        assert fn.__module__ == binding.__name__ and copy.copy(fn) is fn
        assert pickle.loads(pickle.dumps(fn)) is fn
    with pytest.raises(TypeError):
        ng.ngemm_run_u8s8s32(None)
    with pytest.raises(ValueError):
        binding._calls.Call(print, "nothing", 1)


def test_they_are_functions():
    import types
    import weakref
    import paper_1910_00178_amd as ng
    from paper_1910_00178_amd import binding
    fn, plain = ng.ngemm_run_u8s8s32, ng.ngemm_run_u8s8s32.__wrapped__
    assert type(plain) is types.FunctionType and inspect.isfunction(fn) and weakref.ref(fn)() is fn
    assert repr(fn).startswith("<function ngemm_run_u8s8s32 at ")
    for name in ("__code__", "__defaults__", "__globals__", "__kwdefaults__", "__closure__", "__annotations__", "__doc__", "__qualname__", "__module__"):
        assert getattr(fn, name) == getattr(plain, name), name
    assert ng.ngemm_tune_u8s8s32.__doc__ and inspect.getsource(fn) == inspect.getsource(plain)

    class Holder:
        run = fn
    holder = Holder()
    assert inspect.ismethod(holder.run) and holder.run.__self__ is holder and holder.run.__func__ is fn
    with pytest.raises(TypeError):
        holder.run(1, 2)
    fn.note = 5
    assert fn.__dict__.pop("note") == 5
    assert {type(getattr(binding, name)) for name in binding._kinds} == {binding._calls.Call}


def test_collected(both):
    import gc
    import weakref
    call, _, _ = both("run")
    call.itself = call
    gone = weakref.ref(call)
    del call
    gc.collect()
    assert gone() is None


@pytest.mark.parametrize("name", ["_dev", "_stream", "_check"])
def test_a_replaced_name_is_used(both, monkeypatch, name):
    from paper_1910_00178_amd import binding
    call, seen, given = both("run")
    args, _ = usual("run")
    assert call(*args) is None and not given
    with monkeypatch.context() as m:
        m.setattr(binding, name, lambda *a: None)
        assert call(*args) == "slow" and call(*args) == "slow"
    assert call(*args) is None and len(seen) == 2 and len(given) == 2


def test_a_replaced_library_function_is_used(monkeypatch):
    import paper_1910_00178_amd as ng
    from paper_1910_00178_amd import binding
    args, want = usual("run")
    seen = []

    def status(*a):
        seen.append(a)
        return 0
    monkeypatch.setattr(binding._lib, "ngemm_run_u8s8s32", status)
    assert ng.ngemm_run_u8s8s32(*args) is None
    assert [a.value if type(a) is P else a for a in seen[0]] == want
    fake = type("Lib", (), {"ngemm_run_u8u8s32": staticmethod(status)})
    monkeypatch.setattr(binding, "_lib", fake)
    assert ng.ngemm_run_u8u8s32(*args) is None and len(seen) == 2


def test_other_code_defaults_and_stream_lookup(both, monkeypatch):
    from paper_1910_00178_amd import binding
    call, seen, given = both("run")
    args, _ = usual("run")
    monkeypatch.setattr(binding, "_current_stream", lambda: 9)
    binding._calls.streams(lambda d: 0x100 + d, lambda: 7, lambda: True, binding._current_stream)
    assert call(*args[:9]) is None and seen[-1][11] == 0x107
    with monkeypatch.context() as m:
        m.setattr(binding, "_current_stream", lambda: 8)           # asked itself
        assert call(*args[:9]) == "slow" and call(*args) is None
    assert call(*args[:9]) is None
    call.__defaults__ = (1,)
    assert call(*args) == "slow"
    call.__defaults__ = None
    assert call(*args) is None
    code = call.__code__

    def other(*a, **kw):
        return given, "other"
    call.__code__ = other.__code__.replace(co_freevars=code.co_freevars)
    assert call(*args)[1] == "other"
    call.__code__ = code
    assert call(*args) is None


def test_a_profiler_sees_them(both):
    import sys
    call, seen, given = both("run")
    args, _ = usual("run")
    events = []
    sys.setprofile(lambda frame, event, arg: events.append((event, frame.f_code.co_name)))
    try:
        call(*args)
    finally:
        sys.setprofile(None)
    assert ("call", "slow") in events and len(given) == 1 and not seen
    assert call(*args) is None and len(seen) == 1
