"""A call sees what the current stream wrote before it, whichever stream that
is and whether or not its work is done when the call is made: inputs still on
their way on a busy stream (the default one, a side stream, the engine's own),
inputs long there, and a call inside a captured graph."""

import numpy as np
import pytest

from synth import make_events
from tests.gpu_util import torch_cuda, make_engine, run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    torch_cuda()
    import paper_2602_19959_amd as pv
    batch = make_events(4, seed=23)
    eng = make_engine(4, compute_dtype="bf16")
    ref = run(eng, batch)["prob"]
    feat, off = pv.upload_events(batch)
    yield eng, feat, off, ref
    eng.close()


@pytest.mark.parametrize("call", ["execute", "execute_scratch", "graph"])
@pytest.mark.parametrize("where", ["default", "side", "own"])
def test_inputs_still_on_their_way(case, call, where):
    torch = torch_cuda()
    eng, feat, off, ref = case
    s = {"default": torch.cuda.default_stream(), "side": torch.cuda.Stream(), "own": eng.stream}[where]
    late = torch.zeros_like(feat)
    out = eng.alloc_outputs(4)
    torch.cuda.synchronize()
    if call == "graph":
        eng.graph_capture(late, off, out)
    for busy in (True, False, True):
        late.zero_()
        torch.cuda.synchronize()
        print(f"[gpu-stream-order] {call} {where} busy {busy}", flush=True)
        with torch.cuda.stream(s):
            if busy:
                torch.cuda._sleep(20_000_000)        # some ms
            late.copy_(feat)
            if not busy:
                s.synchronize()
            if call == "graph":
                eng.graph_launch()
            else:
                getattr(eng, call)(late, off, out)
        eng.synchronize()
        assert np.array_equal(out.prob.cpu().numpy(), ref)


def test_call_inside_a_captured_graph(case):
    torch = torch_cuda()
    eng, feat, off, ref = case
    late = torch.zeros_like(feat)
    out = eng.alloc_outputs(4)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        late.copy_(feat)
        eng.execute(late, off, out)
        torch.cuda.current_stream().wait_stream(eng.stream)
    for _ in range(3):
        late.zero_()
        out.prob.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.prob.cpu().numpy(), ref)
        got = run(eng, make_events(4, seed=23))["prob"]        # eager work between the replays
        assert np.array_equal(got, ref)
