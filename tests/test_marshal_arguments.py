"""What the native argument marshalling hands to the library, argument by argument.  The extension
module and the ctypes path are both bound to stubs that record every argument of the C ABI - pointer
tables, plans and the update rule by their contents - and return a status of the test's choosing; a
call in a form that the module knows has to be taken by it, and both paths have to pass on the same.
Nothing is launched, so this runs without a GPU.
"""
import ctypes
import types

import numpy as np
import pytest

from paper_1908_04207_amd import binding as eb

if eb._marshal is eb._CtypesOnly:
    pytest.skip("the extension module is not built for this interpreter", allow_module_level=True)

# in the order in which the module is given their addresses
NAMES = ("eager_plan_participation", "eager_plan_quorum", "eager_partial_allreduce_solo",
         "eager_partial_allreduce_majority", "eager_partial_allreduce_quorum",
         "eager_partial_allreduce_lagging", "eager_partial_allreduce_exchange", "eager_sgd_step",
         "eager_sgd_step_lars", "eager_stash", "eager_sgd_step_views", "eager_average_views")
P, BUCKETS = 3, 5
A = 0x10000


class _Buffer:
    """A device buffer as the binding sees one."""
    def __init__(self, p):
        self.p = p

    def data_ptr(self):
        return self.p


class _Stream:
    def __init__(self, p):
        self.cuda_stream = p


def _plan(p):
    return bytes(p.contents)


def _table(n):
    return lambda t: [t[k] for k in range(n)]


def _opt(o):
    return (o.contents.params, o.contents.momentum, o.contents.lr, o.contents.mu) if o else None


def _doubles(n):
    return lambda t: [t[k] for k in range(n)]


def _contents(name, args, sizes):
    """The arguments of a call, what pointers point at in place of the pointers."""
    a = list(args)
    at = {"eager_plan_participation": {2: _doubles(sizes), 7: None}, "eager_plan_quorum": {1: _doubles(sizes), 5: None},
          "eager_partial_allreduce_lagging": {1: _plan, 5: _table(P), 6: _table(P), 8: _opt},
          "eager_partial_allreduce_exchange": {1: _plan, 2: _table(P), 3: _table(P), 5: _opt},
          "eager_sgd_step": {4: _opt}, "eager_sgd_step_lars": {4: _opt}, "eager_stash": {},
          "eager_sgd_step_views": {5: _table(sizes), 6: _table(sizes)}, "eager_average_views": {4: _table(sizes)}}.get(
              name, {1: _plan, 4: _table(P), 5: _table(P), 7: _opt})
    for k, read in at.items():
        a[k] = read(a[k]) if read else "out"
    return a


@pytest.fixture
def stubs(monkeypatch):
    """Both paths bound to recorders.  .calls: (name, arguments); .status: what they return."""
    s = types.SimpleNamespace(calls=[], status=eb.OK)
    real = eb.lib
    keep = []

    def make(name):
        fn = getattr(real, name)

        def record(*args):
            # (sizes that the C side states itself)
            n = {"eager_plan_participation": 1, "eager_plan_quorum": 0, "eager_sgd_step_views": 4,
                 "eager_average_views": 3}.get(name)
            s.calls.append((name, _contents(name, args, args[n] if n is not None else P)))
            if name.startswith("eager_plan"):
                args[-1][0] = eb.Plan(2, 7, 11, 13, 17, 19, 23, 0)
            if name == "eager_partial_allreduce_exchange" and s.status == eb.OK:
                args[2][1], args[3][1] = args[3][1], args[2][1]
            return s.status

        stub = ctypes.CFUNCTYPE(ctypes.c_int, *fn.argtypes)(record)
        keep.append(stub)
        return stub

    fake = types.SimpleNamespace(**{name: getattr(real, name) for name in eb.EXPORTS})
    for name in NAMES:
        setattr(fake, name, make(name))
    monkeypatch.setattr(eb, "lib", fake)
    address = lambda of: tuple(ctypes.cast(getattr(of, n), ctypes.c_void_p).value for n in NAMES)   # noqa: E731
    eb._marshal.bind(address(fake), eb.Plan, ctypes.Array)
    yield s
    eb._marshal.bind(address(real), eb.Plan, ctypes.Array)


class _Taken:
    """The extension module, counting the calls that it takes."""
    def __init__(self, module):
        self.module, self.taken = module, 0

    def __getattr__(self, name):
        fn = getattr(self.module, name)

        def call(*args):
            result = fn(*args)
            self.taken += result is not NotImplemented
            return result
        return call


def _outcome(call):
    try:
        r = call()
        return bytes(r) if isinstance(r, eb.Plan) else r
    except Exception as e:                                  # noqa: BLE001
        return type(e), getattr(e, "status", None), str(e)


def _both(monkeypatch, stubs, call, known=True):
    """The call through the module and through ctypes: the same outcome from the same arguments."""
    module = _Taken(eb._marshal)
    seen = []
    for path in (module, eb._CtypesOnly):
        stubs.calls.clear()
        with monkeypatch.context() as m:
            m.setattr(eb, "_marshal", path)
            outcome = _outcome(call)
        seen.append((outcome, list(stubs.calls)))
    assert seen[0] == seen[1], seen
    assert (module.taken > 0) == known
    if known:
        assert len(seen[0][1]) == 1
    return seen[0]


G, R = [A * (i + 1) for i in range(P)], [A * (i + 9) for i in range(P)]
OPT = (A * 20, A * 21, 0.1, 0.9)
buffers = lambda ptrs: [_Buffer(p) for p in ptrs]                            # noqa: E731
FORMS = [
    dict(), dict(grads=tuple(G), resid=tuple(R)), dict(grads=buffers(G), resid=buffers(R), recv=_Buffer(A * 30)),
    dict(grads=eb.Context.pointers(G), resid=eb.Context.pointers(R)), dict(grads=eb.Context.pointers(G)),
    dict(resid=eb.Context.pointers(buffers(R))), dict(grads=[None, *G[1:]]), dict(resid=[R[0], None, R[2]]),
    dict(recv=None), dict(opt=None), dict(opt=(_Buffer(A * 20), _Buffer(A * 21), 1e-3, 0.0)), dict(opt=(None, None, 1e300, -0.0)),
    dict(b0=1, b1=4), dict(b0=-2, b1=99), dict(b0=3), dict(stream=0), dict(stream=_Stream(A * 40)), dict(stream=_Stream(0)),
    dict(plan=eb.make_plan(eb.QUORUM, P, 1 << 63, 0b110, 2, eb.FLAG_STRICT_QUORUM)), dict(plan=eb.Plan()),
]
OTHER = [dict(opt=list(OPT)), dict(opt=(*OPT[:2], 1, 0.9)), dict(grads=(ctypes.c_int64 * 3)(*G)), dict(grads=G[:2]),
         dict(b0=True), dict(b1=1 << 40), dict(plan=None), dict(grads=[np.int64(3), *G[1:]]), dict(recv=-16),
         dict(recv=1 << 70)]


def _round_arguments(form):
    kw = dict(plan=eb.make_plan(eb.SOLO, P, 6, 0b011, 1), grads=G, resid=R, recv=A * 31, opt=OPT, b0=0, b1=None, stream=A * 41)
    kw.update(form)
    return kw.pop("plan"), kw


@pytest.mark.parametrize("known,form", [(True, f) for f in FORMS] + [(False, f) for f in OTHER])
@pytest.mark.parametrize("status", [eb.OK, eb.ESTATE])
def test_rounds(monkeypatch, stubs, known, form, status):
    stubs.status = status
    plan, kw = _round_arguments(form)
    ctx = eb.Context(P, [64 * b for b in range(BUCKETS)], [60] * BUCKETS)
    for name in ("solo", "majority", "quorum"):
        fn = getattr(ctx, "eager_partial_allreduce_" + name)
        outcome, calls = _both(monkeypatch, stubs, lambda: fn(plan, **kw), known)
        if known:
            ptr = lambda x: x.p if isinstance(x, _Buffer) else x             # noqa: E731
            assert calls[0][0] == "eager_partial_allreduce_" + name
            args = calls[0][1]
            assert args[0] == ctx._addr and args[1] == bytes(plan)
            assert args[2] == kw["b0"] and args[3] == (BUCKETS if kw["b1"] is None else kw["b1"])
            assert args[4] == [ptr(x) for x in kw["grads"]] and args[5] == [ptr(x) for x in kw["resid"]]
            assert args[6] == ptr(kw["recv"]) and (args[7] is None) == (kw["opt"] is None)
            assert (args[8] or 0) == getattr(kw["stream"], "cuda_stream", kw["stream"])
            assert outcome is None if status == eb.OK else outcome[:2] == (eb.EagerError, status)
    for absent in (0, 0b100, 1 << 63, (1 << 64) + 5):
        outcome, calls = _both(monkeypatch, stubs, lambda: ctx.eager_partial_allreduce_lagging(plan, absent, **kw), known)
        if known:
            assert calls[0][1][2] == absent % (1 << 64)
    ctx.close()


@pytest.mark.parametrize("status", [eb.OK, eb.ESTATE])
def test_exchange(monkeypatch, stubs, status):
    """Tables are exchanged in place by the library; lists take the ctypes path."""
    stubs.status = status
    ctx = eb.Context(P, [0], [64])
    plan = eb.make_plan(eb.MAJORITY, P, 2, 0b101)
    for tables in (True, False):
        seen = []
        for opt, recv in ((OPT, None), (None, A * 33), (OPT, _Buffer(A * 34))):
            def call():
                g, r = (eb.Context.pointers(G), eb.Context.pointers(R)) if tables else (list(G), list(R))
                out = None
                try:
                    ctx.eager_partial_allreduce_exchange(plan, g, r, recv=recv, opt=opt, stream=A * 42)
                except eb.EagerError as e:
                    out = e.status
                return out, list(g), list(r)
            outcome, calls = _both(monkeypatch, stubs, call, known=tables)
            assert outcome[0] == (None if status == eb.OK else status)
            late = (R[1], G[1]) if status == eb.OK else (G[1], R[1])
            assert (outcome[1][1], outcome[2][1]) == late and outcome[1][::2] == G[::2] and outcome[2][::2] == R[::2]
            assert calls[0][1][1] == bytes(plan) and calls[0][1][2:4] == [G, R] and calls[0][1][6] == A * 42
    ctx.close()


@pytest.mark.parametrize("status", [eb.OK, eb.EINVAL])
@pytest.mark.parametrize("b0,b1", [(0, None), (1, 3), (-1, 7)])
@pytest.mark.parametrize("stream", [0, A * 43, _Stream(A * 44)])
def test_steps_stash_and_views(monkeypatch, stubs, status, b0, b1, stream):
    stubs.status = status
    ctx = eb.Context(P, [64 * b for b in range(BUCKETS)], [60] * BUCKETS)
    last = BUCKETS if b1 is None else b1
    at = dict(b0=b0, b1=b1, stream=stream)
    raw = getattr(stream, "cuda_stream", stream) or None
    f32 = lambda x: np.float32(x).item()                                     # noqa: E731
    for u in (A, _Buffer(A * 2), None):
        ptr = u.p if isinstance(u, _Buffer) else u
        for opt in (OPT, (_Buffer(A * 5), None, 0.25, 1e-40)):
            fields = (opt[0].p if isinstance(opt[0], _Buffer) else opt[0], opt[1], f32(opt[2]), f32(opt[3]))
            _, calls = _both(monkeypatch, stubs, lambda: ctx.eager_sgd_step(u, opt, **at))
            assert calls == [("eager_sgd_step", [ctx._addr, b0, last, ptr, fields, raw])]
            _, calls = _both(monkeypatch, stubs, lambda: ctx.eager_sgd_step_lars(u, opt, 0.02, 1e-9, **at))
            assert calls == [("eager_sgd_step_lars", [ctx._addr, b0, last, ptr, fields, f32(0.02), f32(1e-9), raw])]
            _both(monkeypatch, stubs, lambda: ctx.eager_sgd_step_lars(u, opt, 1, 1e-9, **at), known=False)
            _both(monkeypatch, stubs, lambda: ctx.eager_sgd_step(u, list(opt), **at), known=False)
        _, calls = _both(monkeypatch, stubs, lambda: ctx.eager_stash(2, u, A * 6, **at))
        assert calls == [("eager_stash", [ctx._addr, 2, b0, last, ptr, A * 6, raw])]
        for w, v in ((G, R), (tuple(G), buffers(R)), (eb.Context.pointers(G), R), (G[:1], R[:1])):
            _, calls = _both(monkeypatch, stubs, lambda: ctx.eager_sgd_step_views(u, w, v, 0.1, 0.9, **at))
            assert calls == [("eager_sgd_step_views", [ctx._addr, b0, last, ptr, len(w), G[:len(w)], R[:len(w)], f32(0.1),
                                                       f32(0.9), raw])]
        _both(monkeypatch, stubs, lambda: ctx.eager_sgd_step_views(u, G, R, 1, 0.9, **at), known=False)
    for views in (G, tuple(buffers(R)), [A] * 64):
        _, calls = _both(monkeypatch, stubs, lambda: ctx.eager_average_views(views, **at))
        assert calls[0][1][:4] == [ctx._addr, b0, last, len(views)] and calls[0][1][5] == raw
        assert calls[0][1][4] == [x.p if isinstance(x, _Buffer) else x for x in views]
    _both(monkeypatch, stubs, lambda: ctx.eager_average_views(eb.Context.pointers(G), **at), known=False)
    ctx.close()


def test_plans(monkeypatch, stubs):
    times = [3.0, float("inf"), -1.5, 2.0]
    for t in (times, tuple(times)):
        for mode, seed, step, window, flags in ((0, 1, 0, 0.0, 0), (1, -5, 1 << 65, 0.5, 1), (7, 1 << 70, -1, -0.0, 0)):
            outcome, calls = _both(monkeypatch, stubs, lambda: eb.eager_plan_participation(mode, t, seed, step, window, flags))
            assert outcome == bytes(eb.Plan(2, 7, 11, 13, 17, 19, 23, 0))
            assert calls == [("eager_plan_participation", [mode, 4, times, seed % (1 << 64), step % (1 << 64), window, flags, "out"])]
        outcome, calls = _both(monkeypatch, stubs, lambda: eb.eager_plan_quorum(t, 3, 9, 0.25))
        assert calls == [("eager_plan_quorum", [4, times, 3, 9, 0.25, "out"])]
    for t in ([1, 2], np.array([1.0, 2.0])):
        _both(monkeypatch, stubs, lambda: eb.eager_plan_participation(0, t, 1, 0), known=False)
    _both(monkeypatch, stubs, lambda: eb.eager_plan_quorum(times, 3, 9, 1), known=False)
    # a refusal comes from ctypes, which says what was refused
    stubs.status = eb.EINVAL
    stubs.calls.clear()
    module = _Taken(eb._marshal)
    with monkeypatch.context() as m:
        m.setattr(eb, "_marshal", module)
        with pytest.raises(eb.EagerError, match="eager_plan_quorum"):
            eb.eager_plan_quorum(times, 3, 9)
    assert module.taken == 1 and [c[0] for c in stubs.calls] == ["eager_plan_quorum"] * 2


def test_current_stream(stubs):
    """No stream given: the current one of the current device, once torch's functions are known."""
    ctx = eb.Context(P, [0], [64])
    asked = []
    eb._marshal.streams(lambda: 3, lambda device: asked.append(device) or A * 50)
    try:
        ctx.eager_stash(1, A, A * 2)
        ctx.eager_sgd_step(A, OPT)
        ctx.eager_partial_allreduce_solo(eb.make_plan(eb.SOLO, P, 0, 1), G, R, opt=OPT)
    finally:
        eb._marshal.streams(None, None)
    assert [args[-1] for _, args in stubs.calls] == [A * 50] * 3 and asked == [3] * 3
    ctx.close()


@pytest.mark.parametrize("name", ["", "_solo", "_majority", "_quorum", "_lagging"])
def test_a_form_that_is_not_known_is_marshalled_once(stubs, monkeypatch, name):
    """A rate that is not exactly a float goes through ctypes; the module is asked about the call once."""
    asked = []

    class Asked:
        def __getattr__(self, fn):
            return lambda *a: asked.append(fn) or getattr(module, fn)(*a)

    module = eb._marshal
    monkeypatch.setattr(eb, "_marshal", Asked())
    ctx = eb.Context(P, [64 * k for k in range(BUCKETS)], [64] * BUCKETS)
    bufs = [A * (k + 1) for k in range(2 * P)]
    absent = [0] if name == "_lagging" else []
    for mode in (eb.SOLO, eb.MAJORITY, eb.QUORUM) if not name else (eb.SOLO,):
        asked.clear(), stubs.calls.clear()
        getattr(ctx, "eager_partial_allreduce" + name)(eb.make_plan(mode, P, 0, 1), *absent, bufs[:P], bufs[P:],
                                                       opt=(A * 20, A * 21, np.float64(0.1), 0.9), stream=0)
        assert asked == ["round"] and len(stubs.calls) == 1
        assert stubs.calls[0][0] == (["eager_partial_allreduce" + name] if name else NAMES[2:5])[0 if name else mode]
    ctx.close()


def test_a_replaced_method_of_a_mode_is_called(stubs, monkeypatch):
    """eager_partial_allreduce goes through the method of the plan's mode where a subclass, the object or the class
    has another than the binding's, with the arguments that the caller gave."""
    seen = []

    class Logged(eb.Context):
        def eager_partial_allreduce_solo(self, plan, grads, resid, **kw):
            seen.append(("solo", plan.step, grads, resid, kw))
            super().eager_partial_allreduce_solo(plan, grads, resid, **kw)

        def eager_partial_allreduce_quorum(self, plan, grads, resid, opt=None):     # takes fewer
            seen.append(("quorum", plan.step, grads, resid, {"opt": opt}))

    def make(cls):
        return cls(P, [64 * k for k in range(BUCKETS)], [64] * BUCKETS)

    G, R = [A * (k + 1) for k in range(P)], [A * (k + 9) for k in range(P)]
    opt = (A * 20, A * 21, 0.1, 0.9)
    ctx = make(Logged)
    ctx.eager_partial_allreduce(eb.make_plan(eb.SOLO, P, 1, 1), G, R, A * 30, opt, 0, 2, 0)
    assert seen == [("solo", 1, G, R, dict(recv=A * 30, opt=opt, b1=2, stream=0))]
    assert [c[0] for c in stubs.calls] == [NAMES[2]] and stubs.calls[0][1][2:4] == [0, 2]
    ctx.eager_partial_allreduce(eb.make_plan(eb.QUORUM, P, 2, 1), G, R, opt=opt)
    assert seen[1:] == [("quorum", 2, G, R, {"opt": opt})] and len(stubs.calls) == 1
    ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, P, 3, 1), G, R, opt=opt, b0=1, stream=0)   # not replaced
    assert len(seen) == 2 and stubs.calls[1][0] == NAMES[3] and stubs.calls[1][1][2:4] == [1, BUCKETS]
    ctx.eager_partial_allreduce_majority = lambda plan, *a, **kw: seen.append((plan.step, a, kw))
    ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, P, 4, 1), G, R, b0=1, b1=1)
    assert seen[2] == (4, (G, R), dict(b0=1, b1=1)) and len(stubs.calls) == 2
    ctx.close()
    plain = make(eb.Context)
    with monkeypatch.context() as m:
        m.setattr(eb.Context, "eager_partial_allreduce_solo", lambda self, plan, *a, **kw: seen.append((plan.step, a, kw)))
        plain.eager_partial_allreduce(eb.make_plan(eb.SOLO, P, 5, 1), G, R)
    assert seen[3] == (5, (G, R), {}) and len(stubs.calls) == 2
    plain.eager_partial_allreduce(eb.make_plan(eb.SOLO, P, 6, 1), G, R, opt=opt, stream=0)
    assert len(seen) == 4 and len(stubs.calls) == 3
    plain.close()
