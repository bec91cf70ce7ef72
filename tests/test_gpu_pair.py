"""enc1's two convolutions in one launch: the bits of the two launches, over
batches that end inside, at and past its 240-row tiles, in both layouts; and
which calls take it."""

import numpy as np
import pytest

from synth import NetShape, make_events
from tests.gpu_util import torch_cuda, make_engine, run

pytestmark = pytest.mark.gpu

PAIR, APART = 42, 28


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("layout", ["event", "interval"])
def test_fused_pair_gives_the_bits_of_two_launches(dtype, layout):
    torch_cuda()
    shape = NetShape(n_levels=3) if layout == "interval" else NetShape()
    batch = make_events(12, seed=23, mix="lognormal")
    eng = make_engine(12, shape=shape, compute_dtype=dtype, unet_layout=layout)
    i = eng.launch_names().index("enc1.c2")
    for n in (1, 2, 5, 12):
        print(f"[gpu-pair] {dtype} {layout} {n} events", flush=True)
        part = batch.subset(range(n))
        got = {}
        for v in (APART, PAIR):
            assert eng.set_variant(i, v)
            fused = eng.launch_kernels()[i - 1] == "conv (in enc1.c2)"
            assert fused == (v == PAIR)
            got[v] = run(eng, part)["prob"], eng.debug_tensor("enc1.c2", n).cpu(), eng.debug_tensor("pool1", n).cpu()
        for a, b in zip(got[APART], got[PAIR]):
            assert np.array_equal(np.asarray(a), np.asarray(b)), n
    eng.close()


def test_conv1_set_by_the_caller_runs_as_set():
    torch_cuda()
    eng = make_engine(2, compute_dtype="bf16")
    i = eng.launch_names().index("enc1.c2")
    assert eng.variants()[i] == PAIR and eng.launch_kernels()[i - 1] == "conv (in enc1.c2)"
    assert eng.set_variant(i - 1, 22)
    assert eng.launch_kernels()[i - 1].startswith("conv_mfma_lp<")
    eng.close()
    # the wide network's enc0.c2 has the same channels but no conv before it: the plain tile
    eng = make_engine(2, shape=NetShape(base_channels=64), compute_dtype="bf16")
    i = eng.launch_names().index("enc0.c2")
    batch = make_events(2, seed=5)
    base = run(eng, batch)["prob"]
    assert eng.set_variant(i, PAIR) and eng.launch_kernels()[i - 1] == "first_conv"
    assert np.array_equal(run(eng, batch)["prob"], base)
    eng.close()
