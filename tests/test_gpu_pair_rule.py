"""Which batches run enc1's two convolutions in one launch, and that the bits do
not depend on it: unset variants on both sides of the rule's lines against the two
launches (set, which pins them), and the second convolution left at its default
under a first one that the caller set."""

import numpy as np
import pytest

from synth import make_events
from tests.gpu_util import torch_cuda, make_engine, run

pytestmark = pytest.mark.gpu

APART = 28
TENSORS = ("enc1.c2", "pool1")


def outputs(eng, batch):
    out = run(eng, batch)
    n = batch.n_events
    return [out["prob"], out["n_vertices"], out["status"]] + [eng.debug_tensor(t, n).cpu().numpy() for t in TENSORS]


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_bits_on_both_sides_of_the_rule(dtype):
    torch = torch_cuda()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows = 2004                                    # of an event at level 1, 240 to a block, 3 blocks to a unit
    eng = make_engine(161, compute_dtype=dtype)
    i = eng.launch_names().index("enc1.c2")
    sizes, fused = (68, 69, 91, 97, 160), {}
    batch = make_events(max(sizes), seed=29, mix="lognormal")
    got = {}
    for n in sizes:
        print(f"[gpu-pair-rule] {dtype} {n} events", flush=True)
        blocks, at_once = -(-n * rows // 240), 3 * cus
        fused[n] = blocks > 2 * at_once or 4 * blocks >= 3 * at_once * -(-blocks // at_once)
        assert (eng.launch_kernels(n)[i - 1] == "conv (in enc1.c2)") == fused[n], n
        got[n] = outputs(eng, batch.subset(range(n)))
    if cus == 256:
        assert [fused[n] for n in sizes] == [False, True, True, False, True]
    assert eng.set_variant(i, APART)
    for n in sizes:
        for a, b in zip(got[n], outputs(eng, batch.subset(range(n)))):
            assert np.array_equal(a, b), n
    eng.close()


def test_first_convolution_set_under_a_default_second():
    torch_cuda()
    n = 90                                         # a batch whose default is the one launch
    batch = make_events(n, seed=31)
    eng = make_engine(n, compute_dtype="bf16")
    i = eng.launch_names().index("enc1.c2")
    want = outputs(eng, batch)
    assert eng.set_variant(i - 1, 22)
    kernels = eng.launch_kernels(n)
    assert kernels[i - 1].startswith("conv_mfma_lp<") and "pair" not in kernels[i]
    for a, b in zip(want, outputs(eng, batch)):
        assert np.array_equal(a, b)
    eng.close()
