"""Which allocator pool the binding's scratch comes from: that of the launch's
own stream, for every form a stream can be named in (no GPU needed)."""

import contextlib

import pytest

torch = pytest.importorskip("torch")
ops = pytest.importorskip("paper_2608_14624_amd.ops",
                          reason="libcachescout.so not built (run __graft_entry__.build())")


@pytest.fixture
def pools(monkeypatch):
    """torch's streams and allocator as a stack of current streams: returns what
    the list of streams that an allocation was made on."""
    current, made_on = ["current"], []

    @contextlib.contextmanager
    def use(stream):
        current.append(stream)
        yield
        current.pop()

    def external(handle, device=None):
        return ("a new stream of torch's pool",) if handle == 0 else ("external", handle)

    monkeypatch.setattr(torch.cuda, "ExternalStream", external)
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device=None: "default")
    monkeypatch.setattr(torch.cuda, "stream", use)
    monkeypatch.setattr(torch, "empty", lambda *a, **k: made_on.append(current[-1]) or "scratch")
    return made_on


@pytest.mark.parametrize("stream,pool", [
    (None, "current"),
    (0, "default"),                       # the null stream
    (1, "default"),                       # the same by its other name
    (1 << 20, ("external", 1 << 20)),
    ("a Stream object", "a Stream object"),
])
def test_scratch_comes_from_the_launch_streams_pool(pools, stream, pool):
    assert ops._scratch(64, stream, "cuda:0") == "scratch"
    assert pools == [pool]


def test_the_per_thread_stream_has_no_pool(pools):
    assert ops._scratch(64, 2, "cuda:0") is None
    assert pools == []
