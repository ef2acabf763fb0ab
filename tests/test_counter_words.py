"""Which stream the counters of inserts and scans are cleared on, without a
GPU: torch is replaced by a stand-in that records it."""

import contextlib
import types

import pytest

from paper_1712_09624_amd import ckpp


class Word:
    def __init__(self, n, stream):
        self.n, self.stream, self.data = n, stream, self

    def split(self, k):
        return tuple(Word(k, self.stream) for _ in range(self.n // k))


@pytest.fixture
def fake(monkeypatch):
    """torch with the current stream `handle` on every device."""
    t = types.SimpleNamespace(handle=0, int64=None, Tensor=Word)
    t.cuda = types.SimpleNamespace(current_device=lambda: 0)
    t._C = types.SimpleNamespace(_cuda_getCurrentRawStream=lambda device: t.handle)
    t.inference_mode = lambda on: contextlib.nullcontext()
    t.zeros = lambda n, dtype=None, device=None: Word(n, t.handle)
    monkeypatch.setattr(ckpp, "_torch", lambda: t)
    monkeypatch.setattr(ckpp, "_zero_words", {})
    return t


DEVICE = types.SimpleNamespace(index=0)


def test_words_of_a_block_are_cleared_on_the_null_stream(fake):
    got = [ckpp._zero_word(DEVICE, 0) for _ in range(ckpp._ZERO_WORDS + 3)]
    assert len({id(w) for w in got}) == len(got)
    assert all(w.n == 1 and w.stream == 0 for w in got)


@pytest.mark.parametrize("current,call", [(7, 0), (0, 7), (7, 7)],
                         ids=["null_call", "null_current", "side"])
def test_no_block_on_another_stream(fake, current, call):
    """A call on the null stream while a side stream is current (and the other
    way round) gets a word of its own, and leaves none for later calls."""
    fake.handle = current
    w = ckpp._zero_word(DEVICE, call)
    assert (w.n, w.stream) == (1, current)
    assert not any(ckpp._zero_words.values())
    fake.handle = 0
    assert ckpp._zero_word(DEVICE, 0).stream == 0


def test_words_are_plain_tensors_of_their_own(monkeypatch):
    """A block made under a tracing mode that hands out stand-ins is not kept
    for later calls, and writing to one word does not look like writing to
    another (autograd's version counter)."""
    import torch
    from torch._subclasses.fake_tensor import FakeTensor, FakeTensorMode
    monkeypatch.setattr(ckpp, "_zero_words", {})
    monkeypatch.setattr(ckpp, "_current_stream_handle", lambda device=None: 0)
    cpu = torch.device("cpu")
    with FakeTensorMode():
        assert isinstance(ckpp._zero_word(cpu, 0), FakeTensor)
    a, b = ckpp._zero_word(cpu, 0), ckpp._zero_word(cpu, 0)
    assert type(a) is type(b) is torch.Tensor and a.shape == b.shape == (1,)
    a.add_(5)
    assert (a.item(), b.item(), b._version) == (5, 0, 0)
