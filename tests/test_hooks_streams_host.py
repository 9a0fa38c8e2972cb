"""Which stream a batch of the saved-tensor hooks is compressed on, without a GPU: the streams and the library's calls are
stand-ins that note what is current.  A tensor that waits for its batch may be written by work on the stream it was saved
on, and its memory goes back to that stream's allocations: it has to be read there, whichever stream is current when the
batch is full or the context ends."""
from __future__ import annotations

import contextlib
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")


class _Streams:
    """Streams of device 0, by number."""

    def __init__(self):
        self.current, self.waits, self.made = 0, [], {}

    def get(self, number):
        if number not in self.made:
            self.made[number] = SimpleNamespace(cuda_stream=number, device_index=0, device=torch.device("cpu"),
                                                wait_stream=lambda other: self.waits.append((number, other.cuda_stream)))
        return self.made[number]

    @contextlib.contextmanager
    def on(self, stream):
        before, self.current = self.current, stream.cuda_stream
        yield
        self.current = before


class _Buffer(SimpleNamespace):
    used_on = ()

    def record_stream(self, stream):
        self.used_on += (stream.cuda_stream,)

    def numel(self):
        return 0

    def element_size(self):
        return 1


@pytest.fixture
def noted(monkeypatch):
    from paper_2510_11400_amd import hooks
    streams, calls, kept = _Streams(), [], {}
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: streams.get(streams.current))
    monkeypatch.setattr(torch.cuda, "stream", streams.on)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: streams.current, raising=False)
    monkeypatch.setattr(hooks.SavedActivations, "_eligible", lambda self, t: True)

    def compress_batch(entries, stream):
        calls.append(("plain", streams.current, [e.tid for e in entries]))

    def compress_channel_wise(xs, splits, k_sigma, share, group_size, bits, rounding, seed, tids):
        calls.append(("routed", streams.current, list(tids)))
        for t in tids:
            kept[t] = SimpleNamespace(data=_Buffer(), nbytes=0)
        return [kept[t] for t in tids]

    def restored(store, dtype):
        calls.append(("restored", streams.current, [t for t in kept if kept[t] is store]))
        return torch.zeros(64, dtype=dtype)

    monkeypatch.setattr(hooks, "api", SimpleNamespace(
        alloc_compressed=lambda *a: (_Buffer(), _Buffer()),
        BatchEntry=lambda g, b, r, s, tid, x, packed, meta: SimpleNamespace(tid=tid, packed=packed, meta=meta),
        Batch=list, fh_compress_batch=compress_batch, compress_channel_wise=compress_channel_wise, restore_channel_wise=restored))
    return SimpleNamespace(hooks=hooks, streams=streams, calls=calls, kept=kept)


@pytest.mark.parametrize("kind", ["plain", "routed"])
def test_a_batch_goes_through_the_streams_its_tensors_were_saved_on(noted, kind):
    h = noted.hooks.SavedActivations(64, 4, min_numel=1, batch_bytes=4 * 64 * 4, channel_dim=0 if kind == "routed" else None)
    for stream in (0, 7, 0, 7):                               # the fourth fills the batch, while stream 7 is current
        noted.streams.current = stream
        h._pack(torch.zeros(8, 8))
    assert noted.calls == [(kind, 0, [0, 2]), (kind, 7, [1, 3])] and not h._pending
    h._pack(torch.zeros(8, 8))                                # and one that the context's end finds waiting
    noted.streams.current = 0
    h.flush()
    assert noted.calls[2:] == [(kind, 7, [4])]
    assert noted.streams.current == 0 and not noted.streams.waits


def test_a_restore_on_another_stream_waits_for_the_batch(noted):
    h = noted.hooks.SavedActivations(64, 4, min_numel=1, batch_bytes=1 << 30, channel_dim=0)
    first, second = h._pack(torch.zeros(8, 8)), h._pack(torch.zeros(8, 8))
    noted.streams.current = 7
    h._unpack(first)                                          # needed back before its batch is full, elsewhere
    assert noted.calls == [("routed", 0, [0, 1]), ("restored", 7, [0])]
    assert noted.streams.waits == [(7, 0)] and noted.kept[0].data.used_on == (7,)
    noted.streams.current = 0
    h._unpack(second)                                         # where it was saved: nothing to wait for
    assert noted.calls[2:] == [("restored", 0, [1])]
    assert noted.streams.waits == [(7, 0)] and noted.kept[1].data.used_on == ()
