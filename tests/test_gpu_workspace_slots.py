"""The kept workspaces of small calls: a workspace must never be in use by two calls at once,
whatever the calls' streams and threads do.  Each case compares calls that share or hand over
workspaces, bit for bit, with the same call run alone: many more streams than slots, one handle
that names another stream in every thread, several threads on one stream, calls of different
shapes and entry points back to back, and a capture between ordinary calls.  The library counts the
calls that ran in a kept workspace, so that each case shows that it reached one."""
import ctypes
import threading

import pytest

import paper_2208_05419_amd as afno
from paper_2208_05419_amd import synth
from gpu_util import dev_weights, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def calls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    made = []
    for i in range(6):
        dtype = "bf16" if i % 2 else "fp32"
        wl = synth.Workload("slots", 1 + i % 2, (24, 45, 60)[i % 3], 60, 64, 2, dtype, 0.01, 1.0)
        w = dev_weights(synth.make_weights(wl, seed=i), dtype)
        x = to_dev(synth.make_x(wl, seed=i), dtype)
        g = to_dev(synth.make_x(wl, seed=100 + i), dtype)
        fwd = lambda x=x, w=w, nb=2: afno.filter_forward(  # noqa: E731
            x, w["w1"], w["b1"], w["w2"], w["b2"], nb, 0.01)
        bwd = lambda x=x, w=w, g=g: afno.filter_backward(  # noqa: E731
            x, w["w1"], w["b1"], w["w2"], w["b2"], g, 2, 0.01)["dx"]
        for f in (fwd, bwd):
            ref = f()
            torch.cuda.synchronize()
            made.append((f, ref.clone()))
    return made


def _same(got):
    torch.cuda.synchronize()
    assert all(torch.equal(a, r) for a, r in got)


def _slot_calls():
    """Calls so far that ran in a kept workspace (afno::g_slot_calls)."""
    return ctypes.c_int64.in_dll(afno.load_library(), "_ZN4afno12g_slot_callsE").value


def test_more_streams_than_slots(calls):
    streams = [torch.cuda.Stream() for _ in range(20)]
    got, n = [], _slot_calls()
    for rep in range(3):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                f, r = calls[(i + rep) % len(calls)]
                got.append((f(), r))
    _same(got)
    assert _slot_calls() >= n + 8


def test_streams_one_after_another(calls):
    """Every stream gets a workspace that an earlier one no longer uses."""
    got, n = [], _slot_calls()
    for i in range(20):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            f, r = calls[i % len(calls)]
            got.append((f(), r))
        s.synchronize()
    _same(got)
    assert _slot_calls() == n + 20


def test_one_handle_for_the_threads_own_streams(calls):
    """hipStreamPerThread (handle 2) is another stream in every thread."""
    got, lock, errors, n = [], threading.Lock(), [], _slot_calls()

    def work(k):
        try:
            s = torch.cuda.ExternalStream(2)
            with torch.cuda.stream(s):
                for i in range(12):
                    f, r = calls[(k + i) % len(calls)]
                    o = f()
                    o.record_stream(s)
                    s.synchronize()
                    with lock:
                        got.append((o.clone(), r))
                s.synchronize()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not errors, errors
    _same(got)
    assert _slot_calls() == n + 48


def test_two_threads_on_one_stream(calls):
    s = torch.cuda.Stream()
    got, lock, errors, n = [], threading.Lock(), [], _slot_calls()

    def work(k):
        try:
            with torch.cuda.stream(s):
                mine = []
                for i in range(20):
                    f, r = calls[(k + i) % len(calls)]
                    mine.append((f(), r))
            with lock:
                got.extend(mine)
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not errors, errors
    _same(got)
    assert _slot_calls() == n + 80


def test_back_to_back_calls_of_different_shapes(calls):
    got, n = [], _slot_calls()
    for rep in range(4):
        for f, r in calls:
            got.append((f(), r))
    _same(got)
    assert _slot_calls() == n + 4 * len(calls)


def test_capture_between_ordinary_calls():
    """A captured call owns its workspace: no kept one is taken, and replays beside ordinary calls
    on the same stream give the ordinary call's bits."""
    wl = synth.Workload("slots", 1, 24, 60, 64, 2, "fp32", 0.01, 1.0)
    w = dev_weights(synth.make_weights(wl, seed=0), "fp32")
    x = to_dev(synth.make_x(wl, seed=0), "fp32")
    args = (w["w1"], w["b1"], w["w2"], w["b2"], 2, 0.01)
    out, s, g = torch.empty_like(x), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        first = afno.filter_forward(x, *args)
    torch.cuda.synchronize()
    n = _slot_calls()
    with torch.cuda.graph(g, stream=s):
        afno.filter_forward(x, *args, out=out)
    assert _slot_calls() == n
    for rep in range(4):
        x.copy_(to_dev(synth.make_x(wl, seed=rep), "fp32"))
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            want = afno.filter_forward(x, *args)
            g.replay()
            again = afno.filter_forward(x, *args)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(again, want)
        assert rep > 0 or torch.equal(want, first)


def test_streams_created_and_destroyed(calls):
    """A stream may be destroyed behind its call: the next stream takes the workspace over, or waits
    for the event where it has the destroyed one's handle."""
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64.so" in line)
    hip = ctypes.CDLL(path)
    hip.hipStreamCreate.argtypes = [ctypes.POINTER(ctypes.c_void_p)]
    hip.hipStreamDestroy.argtypes = [ctypes.c_void_p]
    wl = synth.Workload("slots", 1, 24, 60, 64, 2, "fp32", 0.01, 1.0)
    w = dev_weights(synth.make_weights(wl, seed=0), "fp32")
    x = to_dev(synth.make_x(wl, seed=0), "fp32")
    args = (w["w1"], w["b1"], w["w2"], w["b2"], 2, 0.01)
    want = afno.filter_forward(x, *args)
    outs = [torch.full_like(x, float("nan")) for _ in range(24)]
    torch.cuda.synchronize()
    n = _slot_calls()
    for out in outs:
        h = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(h)) == 0
        afno.filter_forward(x, *args, out=out, stream=torch.cuda.ExternalStream(h.value))
        assert hip.hipStreamDestroy(h) == 0
    _same([(out, want) for out in outs])
    assert _slot_calls() >= n + 8
