"""A child made by fork asks for the stream through the public call again, which refuses a device its parent has initialised:
what the parent found out is not used there."""
import os

import pytest

from paper_2402_04902_amd import binding


@pytest.mark.skipif(not hasattr(os, "fork"), reason="no fork")
def test_forked_child_asks_again(monkeypatch):
    monkeypatch.setattr(binding, "_stream_query", lambda: 0x1234)  # as in a process that has called the library

    def refuse():
        raise RuntimeError("Cannot re-initialize the device in forked subprocess")
    monkeypatch.setattr(binding, "_find_stream_query", refuse)
    assert binding._stream() == 0x1234
    pid = os.fork()
    if pid == 0:
        code = 2
        try:
            binding._stream()
        except RuntimeError:
            code = 0
        except BaseException:
            code = 3
        os._exit(code)
    _, status = os.waitpid(pid, 0)
    assert os.waitstatus_to_exitcode(status) == 0
    assert binding._stream() == 0x1234
