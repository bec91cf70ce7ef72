"""A call on one thread while another thread has a stream capture open, in the
capture modes that forbid unsafe calls on the capturing thread or on every thread:
the call is made, its results are its own, and the other thread's graph is whole."""

import threading

import numpy as np
import pytest

from synth import make_events
from tests.gpu_util import torch_cuda, make_engine, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["thread_local", "global"])
@pytest.mark.parametrize("busy", [False, True])
def test_call_beside_another_threads_capture(mode, busy):
    torch = torch_cuda()
    import paper_2602_19959_amd as pv
    batch = make_events(4, seed=23)
    eng = make_engine(4, compute_dtype="bf16")
    ref = run(eng, batch)["prob"]
    feat, off = pv.upload_events(batch)
    out = eng.alloc_outputs(4)
    x = torch.ones(1024, device="cuda")
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    opened, go, graph = threading.Event(), threading.Event(), torch.cuda.CUDAGraph()
    failed = []

    def capture():
        try:
            with torch.cuda.graph(graph, stream=torch.cuda.Stream(), capture_error_mode=mode):
                y.copy_(x)
                opened.set()
                go.wait(20)
                y.add_(1)
        except Exception as e:                      # told to the test, which would else wait
            failed.append(e)
            opened.set()

    t = threading.Thread(target=capture)
    t.start()
    assert opened.wait(20)
    try:
        if busy:
            torch.cuda._sleep(5_000_000)
        eng.execute(feat, off, out)
    finally:
        go.set()
        t.join()
    assert not failed
    graph.replay()
    torch.cuda.synchronize()
    assert bool((y == 2).all())
    assert np.array_equal(out.prob.cpu().numpy(), ref)
    eng.close()
