"""Scratch calls of four live engines in flight together, each on its own stream
without any order between them, give the bits of each call alone; also after
engines were destroyed and others took their areas."""

import numpy as np
import pytest

from synth import make_events
from tests.gpu_util import torch_cuda, engine_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n", [("fp32", 8), ("fp8_e4m3", 35)])
def test_scratch_calls_of_four_engines_overlap(dtype, n):
    torch = torch_cuda()
    import paper_2602_19959_amd as pv
    batches = [pv.upload_events(make_events(n, seed=40 + k)) for k in range(4)]
    engines = [engine_for(n, dtype) for _ in range(4)]
    for turn in range(2):
        outs = [e.alloc_outputs(n) for e in engines]
        alone = []
        for e, b in zip(engines, batches):
            e.execute(*b, outs[0])
            e.synchronize()
            alone.append(outs[0].prob.cpu().numpy())
        torch.cuda.synchronize()
        print(f"[gpu-scratch-areas] {dtype} turn {turn}", flush=True)
        for _ in range(10):
            for e, b, o in zip(engines, batches, outs):
                e.execute_scratch(*b, o)
        torch.cuda.synchronize()
        for k, o in enumerate(outs):
            assert np.array_equal(o.prob.cpu().numpy(), alone[k]), (turn, k)
        # two engines go, two others take their areas
        for k in (1, 2):
            engines[k].close()
            engines[k] = engine_for(n, dtype)
    for e in engines:
        e.close()
