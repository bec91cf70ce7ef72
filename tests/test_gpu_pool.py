"""The pooled tensors are the maxima of the stored row pairs, exactly: FP8
compares codes, the other types values."""

import numpy as np
import pytest

from synth import make_events
from tests.gpu_util import torch_cuda, engine_for, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp16", "fp8_e4m3"])
@pytest.mark.parametrize("events", [1, 3, 40])
def test_pooled_rows_are_pair_maxima(dtype, events):
    torch_cuda()
    eng = engine_for(40, dtype)
    run(eng, make_events(events, seed=31, mix="lognormal"))
    for l, c in ((0, 32), (1, 64), (2, 128)):
        full = eng.debug_tensor(f"enc{l}.c2", events).cpu().numpy().reshape(events, c, 4000 >> l)
        pool = eng.debug_tensor(f"pool{l}", events).cpu().numpy().reshape(events, c, 2000 >> l)
        assert np.array_equal(full.reshape(events, c, -1, 2).max(-1), pool), (dtype, events, l)
    eng.close()
