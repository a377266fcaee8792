"""The timing helpers make their first calls on a stream of their own: that
stream waits for the current one first, where the inputs are made and the
workspaces zero-filled (no GPU: the stream calls are recorded)."""

import contextlib
import os
import sys

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402
from paper_2411_12692_amd import schedule  # noqa: E402


class _Stop(Exception):
    pass


@pytest.mark.parametrize("helper", [lambda fn: bench.time_steps(fn, 4, 2), lambda fn: bench.graph_us(fn, 2),
                                    lambda fn: schedule._graph_time_us([lambda: fn(0)], 1)],
                         ids=["time_steps", "graph_us", "schedule"])
def test_first_call_waits_for_the_current_stream(monkeypatch, helper):
    log = []

    class Stream:
        def wait_stream(self, other):
            log.append(("wait", other))

    def stop():
        raise _Stop

    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: "current")
    monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())
    monkeypatch.setattr(torch.cuda, "synchronize", stop)  # the helpers synchronize once their first calls are made
    with pytest.raises(_Stop):
        helper(lambda i: log.append(("call", i)))
    assert log[0] == ("wait", "current") and log[1][0] == "call"
