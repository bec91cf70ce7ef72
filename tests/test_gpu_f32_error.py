"""The error of p against FP64 is no larger than with FP32 matrix instructions:
per network and events, the relative 2-norm over two events measured once with
v_mfma_f32_16x16x4_f32 convolutions is the bar.  Seeds 2, 13, 14 and, of the
64-channel networks, 20 are those of 64 where one accumulator chain of all six
BF16 products was less accurate."""

import numpy as np
import pytest

import oracle
from synth import NetShape, make_events
from tests.gpu_util import blob, run, torch_cuda, weights

pytestmark = pytest.mark.gpu

# (width, seed): error with the FP32 instruction
FP32_INSTRUCTION = {(32, 0): 1.971e-7, (32, 2): 4.358e-7, (32, 13): 1.108e-7, (32, 14): 3.189e-7,
                    (64, 1): 7.826e-7, (64, 20): 4.783e-7}


@pytest.mark.parametrize("width,seed", sorted(FP32_INSTRUCTION))
def test_error_is_not_above_the_fp32_instructions(width, seed):
    torch_cuda()
    import paper_2602_19959_amd as pv
    shape = NetShape(base_channels=width)
    batch = make_events(2, seed=seed + 100)
    eng = pv.Engine(blob(seed, shape), pv.default_spec(max_events=2, max_tracks_total=3000, base_channels=width))
    p = run(eng, batch)["prob"].astype(np.float64)
    eng.close()
    ref = np.stack([r["p"] for r in oracle.run_batch(batch, weights(seed, shape))])
    error = np.linalg.norm(p - ref) / np.linalg.norm(ref)
    print(f"[gpu-f32-error] width {width} seed {seed}: {error:.2e} of {FP32_INSTRUCTION[width, seed]:.2e}", flush=True)
    assert error <= FP32_INSTRUCTION[width, seed]
