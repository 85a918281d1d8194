"""Threads that call the library beside a thread that captures a graph: what the library keeps per thread is given back when
the thread ends, which must not disturb the capture."""
import threading
import time

import pytest
import torch

from paper_2311_10359_amd import binding, traces
from parity_util import DEV

pytestmark = pytest.mark.gpu


def test_a_thread_ends_while_another_captures():
    rec, off = traces.build(traces.config(0))
    d_rec, d_off = binding.to_device_records(rec, DEV), binding.to_device_u64(off, DEV)
    want = binding.fikit_profile(d_rec, d_off)
    called, may_end, rows = threading.Event(), threading.Event(), []

    def work():
        rows.append(binding.fikit_profile(d_rec, d_off).n_rows)
        called.set()
        may_end.wait(60)

    thread = threading.Thread(target=work)
    thread.start()
    assert called.wait(60)
    x = torch.zeros(1000, device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="global"):
        x.add_(1)
        may_end.set()
        thread.join(60)
        time.sleep(0.5)      # (a thread's own variables go after Python has let go of it)
        x.add_(1)
    for _ in range(3):
        graph.replay()
    torch.cuda.synchronize()
    assert rows == [want.n_rows] and torch.equal(x, torch.full_like(x, 6))
