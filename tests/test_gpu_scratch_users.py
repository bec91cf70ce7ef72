"""Only engines that make scratch calls take a scratch area, and an area is free
for the next engine once the work on it is done: scratch calls in flight together
give the bits of each call alone, with engines made between them that never use
the scratch, and after an engine was destroyed with its calls still queued."""

import numpy as np
import pytest

from synth import make_events
from tests.gpu_util import torch_cuda, engine_for

pytestmark = pytest.mark.gpu

N = 8


def alone(engines, batches):
    want = []
    for e, b in zip(engines, batches):
        out = e.alloc_outputs(N)
        e.execute(*b, out)
        e.synchronize()
        want.append(out.prob.cpu().numpy())
    return want


def test_engines_without_scratch_calls_take_no_area():
    torch = torch_cuda()
    import paper_2602_19959_amd as pv
    batches = [pv.upload_events(make_events(N, seed=60 + k)) for k in range(4)]
    users = [engine_for(N, "fp32")]
    plain = []
    for _ in range(3):                       # three engines without scratch calls before each further user
        plain += [engine_for(N, "fp32") for _ in range(3)]
        users.append(engine_for(N, "fp32"))
    want = alone(users, batches)
    outs = [e.alloc_outputs(N) for e in users]
    torch.cuda.synchronize()
    print("[gpu-scratch-users] four users among nine others", flush=True)
    for _ in range(10):
        for e, b, o in zip(users, batches, outs):
            e.execute_scratch(*b, o)
    torch.cuda.synchronize()
    for k, o in enumerate(outs):
        assert np.array_equal(o.prob.cpu().numpy(), want[k]), k
    for e in users + plain:
        e.close()


def test_area_is_given_back_after_the_work_on_it():
    torch = torch_cuda()
    import paper_2602_19959_amd as pv
    batches = [pv.upload_events(make_events(N, seed=70 + k)) for k in range(2)]
    others = [engine_for(N, "fp32") for _ in range(3)]       # hold the other three areas
    for e in others:
        e.execute_scratch(*batches[0])
    first, second = engine_for(N, "fp32"), engine_for(N, "fp32")
    want = alone([first, second], batches)
    o1, o2 = first.alloc_outputs(N), second.alloc_outputs(N)
    torch.cuda.synchronize()
    with torch.cuda.stream(first.stream):
        torch.cuda._sleep(20_000_000)                        # some ms, then the call
    for _ in range(5):
        first.execute_scratch(*batches[0], o1)
    assert first.lib.pvf_destroy(first.handle) == 0          # without close()'s own wait
    first.handle = None
    print("[gpu-scratch-users] area reused after destroy", flush=True)
    second.execute_scratch(*batches[1], o2)
    torch.cuda.synchronize()
    assert np.array_equal(o1.prob.cpu().numpy(), want[0]) and np.array_equal(o2.prob.cpu().numpy(), want[1])
    for e in others + [second]:
        e.close()
