"""Whose scratch a call without workspace= takes: calls of two streams, of two threads or of a graph and its replays never meet in one buffer."""
import threading

import pytest
import torch

from paper_1412_4564_amd import binding as B


CPU = torch.device("cpu")


def _on_stream(monkeypatch, handle, capturing=False):
    monkeypatch.setattr(B, "_stream", lambda: handle)
    monkeypatch.setattr(B, "_capturing", lambda: capturing)


def _get(nbytes):
    ptr, n, stream = B._scratch(None, nbytes, CPU)
    assert stream == B._stream()
    return ptr, n


def _in_thread(f):
    got = []
    t = threading.Thread(target=lambda: got.append(f()))
    t.start()
    t.join()
    return got[0]


def test_buffers_by_stream_and_thread(monkeypatch):
    monkeypatch.setattr(B, "_default_ws", type(B._default_ws)())
    _on_stream(monkeypatch, 1)
    a = _get(1000)
    assert _get(1000) == a and _get(400) == a                  # one stream: the same buffer
    _on_stream(monkeypatch, 2)
    b = _get(1000)
    assert abs(b[0] - a[0]) >= 1000
    assert _in_thread(lambda: _get(1000))[0] not in (a[0], b[0])      # both of this thread are still held
    grown = _get(5000)
    assert grown[1] >= 5000 and _get(1000) == grown
    _on_stream(monkeypatch, 1)
    assert _get(1000) == a                                            # another stream's growth leaves it alone
    assert _get(0) == (None, 0)


def test_buffers_are_bounded(monkeypatch):
    monkeypatch.setattr(B, "_default_ws", type(B._default_ws)())
    for handle in range(1, 100):
        _on_stream(monkeypatch, handle)
        _get(1000)
    assert len(B._default_ws.bufs) <= B._default_ws.MOST


def test_graph_leaves_the_kept_buffers_alone(monkeypatch):
    monkeypatch.setattr(B, "_default_ws", type(B._default_ws)())
    _on_stream(monkeypatch, 1)
    a = _get(1000)
    _on_stream(monkeypatch, 1, capturing=True)
    for nbytes in (1000, 100000):
        assert _get(nbytes)[0] != a[0]
    _on_stream(monkeypatch, 1)
    assert _get(1000) == a


@pytest.mark.parametrize("gone", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_without_the_private_names(monkeypatch, gone):
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0)
    monkeypatch.delattr(torch._C, gone)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("Stream", (), {"cuda_stream": 77}))
    assert B._stream() == 77


# Input derivatives of strided layers (packed weights of four phases and shared tiles in scratch) and bias derivatives (partial sums).
LAYERS = [((4, 64, 48, 48), (256, 64, 6, 6), (2, 2), (2, 2, 2, 2)), ((3, 40, 20, 23), (70, 40, 3, 3), (2, 2), (1, 0, 0, 1)),
          ((2, 96, 30, 28), (128, 96, 3, 3), (1, 1), (1, 1, 1, 1)), ((5, 48, 33, 41), (80, 48, 5, 4), (2, 3), (0, 1, 1, 0))]


def _passes(layer, seed):
    xs, ws, st, pad = LAYERS[layer]
    g = torch.Generator(device="cuda").manual_seed(seed)
    x, w = (torch.randn(s, device="cuda", generator=g) for s in (xs, ws))
    p = torch.randn(B.conv_forward(x, w, None, st, pad).shape, device="cuda", generator=g)

    def run():
        return (B.conv_forward(x, w, None, st, pad), B.conv_backward_data(xs, w, p, st, pad), B.conv_backward_filter(x, ws, p, st, pad),
                B.conv_backward_bias(xs, ws, p, st, pad))
    return run


@pytest.mark.gpu
@pytest.mark.parametrize("threads", [False, True])
def test_two_streams_at_once(threads):
    """Every result bit for bit that of the calls one after the other."""
    runs = [_passes(i, 10 + i) for i in range(len(LAYERS))]
    want = [r() for r in runs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in runs]
    print("streams at once", threads, flush=True)
    got = [[] for _ in runs]

    def work(i, rounds):
        with torch.cuda.stream(streams[i]):
            for _ in range(rounds):
                got[i].append(runs[i]())

    if threads:
        ts = [threading.Thread(target=work, args=(i, 20)) for i in range(len(runs))]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
    else:
        for _ in range(20):
            for i in range(len(runs)):
                work(i, 1)
    torch.cuda.synchronize()
    for i, results in enumerate(got):
        assert len(results) == 20
        for r in results:
            assert all(torch.equal(a, b) for a, b in zip(r, want[i])), LAYERS[i]


@pytest.mark.gpu
def test_graph_beside_eager_calls():
    """Replays of a graph that took its scratch itself, beside eager calls of more scratch on another stream."""
    small, large = _passes(1, 5), _passes(0, 6)
    want, wantl = small(), large()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        got = small()
    side = torch.cuda.Stream()
    print("graph beside eager calls", flush=True)
    for _ in range(5):
        for t in got:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            eager = large()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        assert all(torch.equal(a, b) for a, b in zip(eager, wantl))
