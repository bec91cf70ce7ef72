"""Only engines that make scratch calls take a scratch area: scratch calls in
flight together give the bits of each call alone, with engines made between them
that never use the scratch."""

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
