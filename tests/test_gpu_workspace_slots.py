"""The kept workspaces of small calls: a workspace must never be in use by two calls at once,
whatever the calls' streams and threads do.  Each case compares calls that share or hand over
workspaces, bit for bit, with the same call run alone: many more streams than slots, one handle
that names another stream in every thread, several threads on one stream, and calls of different
shapes and entry points back to back."""
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


def test_more_streams_than_slots(calls):
    streams = [torch.cuda.Stream() for _ in range(20)]
    got = []
    for rep in range(3):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                f, r = calls[(i + rep) % len(calls)]
                got.append((f(), r))
    _same(got)


def test_one_handle_for_the_threads_own_streams(calls):
    """hipStreamPerThread (handle 2) is another stream in every thread."""
    got, lock, errors = [], threading.Lock(), []

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


def test_two_threads_on_one_stream(calls):
    s = torch.cuda.Stream()
    got, lock, errors = [], threading.Lock(), []

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


def test_back_to_back_calls_of_different_shapes(calls):
    got = []
    for rep in range(4):
        for f, r in calls:
            got.append((f(), r))
    _same(got)
