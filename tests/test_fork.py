"""A forked child of a process that has used the GPU must not launch with the parent's runtime: torch refuses there, and
the binding's short way to the current stream must not pass that refusal by.  Host only."""
import os

from paper_1808_05567_amd import conv


def test_a_forked_child_asks_torch_for_its_stream_again(monkeypatch):
    monkeypatch.setattr(conv, "_raw_stream", lambda: 1234)  # (as after the first call on a GPU)
    assert conv._stream(None) == 1234
    pid = os.fork()
    if pid == 0:
        os._exit(0 if conv._raw_stream is None else 1)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
    assert conv._stream(None) == 1234
