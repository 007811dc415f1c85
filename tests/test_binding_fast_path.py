"""The binding's way for ordinary tensors gives the C entry what the general way gives it, or leaves the call to it, for
every form of a call (no GPU: a class that answers like a tensor stands in for torch's).
"""
import itertools

import pytest

import paper_1305_4376_amd as td


class Device:
    type = "cuda"


class Tensor:
    """What the binding asks of a tensor."""

    device = Device()

    def __init__(self, address, nbytes, contiguous=True, index=0):
        self.address, self.nbytes, self.contiguous, self.index = address, nbytes, contiguous, index

    def get_device(self):
        return self.index

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return self.address

    def numel(self):
        return self.nbytes

    def element_size(self):
        return 1


class Other(Tensor):
    """A tensor of another class goes the general way."""


class Stream:
    cuda_stream = 77


CURRENT = 55  # the current stream of every device here


@pytest.fixture(autouse=True)
def stand_in(monkeypatch):
    general = td._stream
    monkeypatch.setattr(td, "_torch_fast", (Tensor, lambda index: CURRENT))
    monkeypatch.setattr(td, "_stream", lambda stream, like=None: CURRENT if stream is None else general(stream))


def _outcome(kind, sched, src, dst, n, stream):
    make = [kind(address, *form) for address, form in ((1000, sched), (2000, src), (3000, dst))]
    try:
        return td._message_args(*make, n, stream)
    except ValueError as e:
        return str(e)


SCHEDS = [(1600,), (1599,), (3200,), (1600, False)]
SOURCES = [(64,), (0,), (60,), (68,), (64, False), (64, True, -1)]
TARGETS = [(64,), (56,), (72,), (64, False)]
COUNTS = [None, 0, 1, 8, 9, -1, True, 8.0]
STREAMS = [None, 0, 12, Stream()]


def test_both_ways_agree():
    for form in itertools.product(SCHEDS, SOURCES, TARGETS, COUNTS, STREAMS):
        assert _outcome(Tensor, *form) == _outcome(Other, *form), form


@pytest.mark.parametrize("stream", STREAMS)
@pytest.mark.parametrize("n", [None, 8])
def test_ordinary_calls_do_not_go_the_general_way(monkeypatch, n, stream):
    monkeypatch.setattr(td, "_nblocks", None)
    want = (1000, 2000, 3000, 8, CURRENT if stream is None else getattr(stream, "cuda_stream", stream))
    assert _outcome(Tensor, (1600,), (64,), (64,), n, stream) == want
