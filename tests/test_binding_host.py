"""The Python binding where it keeps something between calls; no GPU."""
import os

from paper_2511_04002_amd import tsq


def test_a_forked_child_asks_torch_for_the_stream_again(monkeypatch):
    """torch refuses to use a device in a forked child of a process that has used it; the accessor that the parent
    found does not, so the child must not inherit it."""
    monkeypatch.setattr(tsq, "_current_stream", lambda: 0)
    assert tsq.Plan._stream() == 0
    child = os.fork()
    if child == 0:
        os._exit(0 if tsq._current_stream is None else 1)
    assert os.waitstatus_to_exitcode(os.waitpid(child, 0)[1]) == 0
    assert tsq._current_stream is not None
