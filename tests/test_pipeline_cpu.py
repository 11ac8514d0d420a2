"""SparseStack's host logic without a GPU: the calls of its methods on a stack
whose native executor and streams are stand-ins."""
import contextlib

import pytest
import torch

from paper_2608_09388_amd import pipeline


@pytest.mark.parametrize("device", [0, 1])
def test_step_runs_on_the_stacks_device(monkeypatch, device):
    """The native loop refuses a current device that is not the stack's, so
    step() calls it with the stack's stream, and so its device, current where
    another device is."""
    current = [None]

    @contextlib.contextmanager
    def stream(s):
        before, current[0] = current[0], s
        try:
            yield
        finally:
            current[0] = before

    class Main:
        device_index = 0

    monkeypatch.setattr(torch.cuda, "stream", stream)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: device)
    main = Main()
    seen = []

    class Native:
        def run(self, steps, stream, feed=None, time_layer=0, time_events=None, cur_set=0,
                prev_rows=0):
            seen.append((current[0], stream is main, steps, cur_set, prev_rows))
            return 42, 1, 7

    class Set:
        n = None

    st = pipeline.SparseStack.__new__(pipeline.SparseStack)
    st._native, st.side, st.main, st._one_device = Native(), None, main, False
    st._sets, st._cur, st.prev_n = [Set(), Set()], 0, 3
    st._enter, st._leave = (lambda: None), (lambda cur: None)
    assert st.step() == 42
    assert seen == [(main if device == 1 else None, True, 1, 0, 3)]
    assert st._cur == 1 and st.prev_n == 7 and st.n == 42
    assert current == [None]
