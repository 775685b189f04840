"""LSTM layers of several streams and threads: their sequence launches take turns on the
device, and a layer waits for nothing that another stream has only queued."""
import threading

import numpy as np
import pytest

from tests._gpu import darb, dev, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu

H, T, B = 256, 40, 16


@pytest.fixture(scope="module")
def layer(darb):  # noqa: F811
    rng = np.random.default_rng(3)
    mats = []
    for n in (64, H):
        d = np.clip(0.06 * rng.lognormal(0.0, 0.5, size=4 * H), 0.0, 1.0)
        plan = darb.Plan(4 * H, n, d, 0.06, 0, 4, 64).upload()
        W = (0.1 * rng.standard_normal((4 * H, n))).astype(np.float16)
        mats.append((plan,) + plan.encode(dev(W)))
    x = [dev(rng.standard_normal((64, T * B)).astype(np.float32)) for _ in range(4)]
    run = lambda i, **k: darb.lstm_layer(mats[0], mats[1], x[i], H, T, B, **k)  # noqa: E731
    want = [run(i) for i in range(4)]
    torch.cuda.synchronize()
    return run, want


def _independent_streams(cycles):
    """A stream kept busy by a sleep kernel, and one whose work runs meanwhile."""
    a = torch.cuda.Stream()
    small = torch.zeros(16, device="cuda")
    torch.cuda.synchronize()
    for _ in range(8):                                   # some share a hardware queue
        b = torch.cuda.Stream()
        done = torch.cuda.Event()
        with torch.cuda.stream(a):
            torch.cuda._sleep(cycles)
            done.record()
        with torch.cuda.stream(b):
            small.add_(1.0)
        b.synchronize()
        free = not done.query()
        torch.cuda.synchronize()
        if free:
            return a, b
    pytest.skip("no two streams on queues of their own")


def test_layer_does_not_wait_for_a_queued_one(darb, layer):  # noqa: F811
    # stream a has a layer queued behind other work (here a kernel of some 0.1 s); stream
    # b's layer, called later, ends before that work does.  If it waited, and that work for
    # its results, neither would ever end.
    run, want = layer
    cycles = 200_000_000
    a, b = _independent_streams(cycles)
    say("lstm layer beside a queued one")
    done = torch.cuda.Event()
    with torch.cuda.stream(a):
        torch.cuda._sleep(cycles)
        done.record()
        first = run(0)
    with torch.cuda.stream(b):
        second = run(1)
    b.synchronize()
    assert not done.query()
    torch.cuda.synchronize()
    for got, w in ((first, want[0]), (second, want[1])):
        for g, e in zip(got, w):
            assert torch.equal(g, e)


class _PerThreadDefault:
    """hipStreamPerThread: one handle, a stream of its own for every host thread."""
    cuda_stream = 2


@pytest.mark.parametrize("streams", ["own", "per_thread_default"])
def test_layers_of_several_threads(darb, layer, streams):  # noqa: F811
    run, want = layer
    say(f"lstm layers of four threads, streams: {streams}")
    bufs = [dict(h=torch.empty(H, B, device="cuda"), c=torch.empty(H, B, device="cuda"),
                 h_seq=torch.empty(H, T * B, device="cuda"),
                 workspace=torch.empty(darb.lstm_workspace_floats(H, T, B), device="cuda"))
            for _ in range(4)]
    own = [torch.cuda.Stream() for _ in range(4)]
    bad, errors = [], []
    start = threading.Barrier(4, timeout=30)

    def work(i):
        try:
            s = own[i] if streams == "own" else _PerThreadDefault
            start.wait()
            for _ in range(10):
                # the state is cleared for the whole device before the next call
                bufs[i]["h"].zero_()
                bufs[i]["c"].zero_()
                torch.cuda.synchronize()
                run(i, stream=s, **bufs[i])
                torch.cuda.synchronize()
                if not all(torch.equal(bufs[i][k], w)
                           for k, w in zip(("h_seq", "h", "c"), want[i])):
                    bad.append(i)
        except Exception as e:                            # noqa: BLE001
            errors.append(e)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors and not bad
