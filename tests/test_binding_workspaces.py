"""Scratch of the Python binding: never shared by calls that are not ordered on one stream, bounded, and kept while a
captured graph may refer to it.  The table is host code; it runs here on CPU tensors with made-up stream handles."""
import contextlib
import threading

import pytest
import torch

from paper_2605_16154_amd import binding

CPU = torch.device("cpu")


@pytest.fixture(autouse=True)
def empty_table(monkeypatch):
    monkeypatch.setattr(binding, "_workspaces", {})
    monkeypatch.setattr(binding, "_captured_workspaces", {})
    monkeypatch.setattr(binding, "_capturing", lambda: False)


@contextlib.contextmanager
def take(nbytes, stream):
    """What a call does around its launches."""
    ws = binding._take_workspace(nbytes, CPU, stream)
    try:
        yield ws
    finally:
        binding._give_workspace(ws, CPU, stream)


def test_one_stream_reuses_its_scratch_and_two_streams_have_their_own():
    with take(1000, 0) as a:
        first = a.data_ptr()
    with take(500, 0) as b:
        assert b.data_ptr() == first and b.numel() == 1000
    with take(1000, 7) as c:
        assert c.data_ptr() != first
        other = c.data_ptr()
    with take(1000, 0) as d, take(1000, 7) as e:
        assert (d.data_ptr(), e.data_ptr()) == (first, other)
    with take(2000, 0) as f:
        assert f.numel() == 2000
    with take(1000, 0) as g:
        assert g.numel() == 2000


def test_calls_that_issue_at_the_same_time_on_one_stream_have_their_own():
    with take(1000, 0):
        pass
    inside, out = threading.Barrier(4, timeout=30), []

    def call():
        with take(1000, 0) as w:
            inside.wait()                  # all four are between taking and giving back
            out.append(w.data_ptr())
            inside.wait()

    threads = [threading.Thread(target=call) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(set(out)) == 4
    assert len(binding._workspaces) == 1


def test_table_is_bounded_and_drops_what_was_used_longest_ago():
    for stream in range(binding._KEPT_WORKSPACES):
        with take(100, stream):
            pass
    with take(100, 0):                     # used again: no longer the oldest
        pass
    with take(100, 1000):
        pass
    assert len(binding._workspaces) == binding._KEPT_WORKSPACES
    assert (None, 0) in binding._workspaces and (None, 1) not in binding._workspaces


def test_scratch_of_a_capture_is_the_graphs_from_then_on(monkeypatch):
    """The graph may be replayed on any stream at any later time: neither eager calls on the capture's stream nor growth
    nor the bound of the table may touch its scratch.  Later captures on the stream take it again, or a larger one."""
    with take(300, 3) as w:                # warm-up: sizes the scratch before the capture
        warm = w
    monkeypatch.setattr(binding, "_capturing", lambda: True)
    with take(0, 3) as v, take(100, 3) as w:
        assert v is warm and w is warm     # calls of one capture are ordered: one tensor serves them
    monkeypatch.setattr(binding, "_capturing", lambda: False)
    with take(100, 3) as w:
        assert w is not warm
    monkeypatch.setattr(binding, "_capturing", lambda: True)
    with take(200, 3) as w:
        assert w is warm
    with take(400, 3) as w:
        larger = w
        assert w.numel() >= 400
    with take(100, 3) as w:
        assert w is larger
    assert [c is t for c, t in zip(binding._captured_workspaces[(None, 3)], (warm, larger))] == [True, True]
    monkeypatch.setattr(binding, "_capturing", lambda: False)
    assert not any(t is c for t in binding._workspaces.values() for c in (warm, larger))


def test_an_error_in_the_call_gives_the_scratch_back():
    with pytest.raises(binding.PcmError):
        with take(100, 0):
            raise binding.PcmError("refused")
    assert len(binding._workspaces) == 1
