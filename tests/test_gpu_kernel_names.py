"""The kernels that launch_kernels(n) reports are those that a call of n events
launches, in order: recorded by the GPU's own trace, at batch sizes that run small
tiles, that run enc1's two convolutions apart and in one launch, and larger ones.
The trace's demangler does not know the 16-bit types, so the template arguments
are compared in FP32 and FP8 only."""

import re

import pytest

from synth import make_events
from tests.gpu_util import torch_cuda, engine_for

pytestmark = pytest.mark.gpu


def traced(torch, eng, feat, off, out):
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        eng.execute(feat, off, out)
        torch.cuda.synchronize()
    ours = [e for e in prof.events() if "3pvf" in e.name or "pvf::" in e.name]
    return [e.name for e in sorted(ours, key=lambda e: e.time_range.start)]


def base(name):
    return re.search(r"(track_stage_mma|first_conv|peak_finder|conv_mfma_[a-z0-9_]+?)(?=I[DLhf]|<|$)", name).group(1)


def arguments(name):
    return re.search(r"<(.*?)>(\(pvf::|$)", name).group(1).replace(" ", "")


@pytest.mark.parametrize("dtype,sizes", [("fp32", (1, 40)), ("bf16", (2, 90, 97)), ("fp16", (1,)),
                                         ("fp8_e4m3", (1, 60))])
def test_reported_kernels_are_the_launched_ones(dtype, sizes):
    torch = torch_cuda()
    import paper_2602_19959_amd as pv
    eng = engine_for(max(sizes), dtype)
    for n in sizes:
        feat, off = pv.upload_events(make_events(n, seed=3))
        out = eng.alloc_outputs(n)
        eng.execute(feat, off, out)
        torch.cuda.synchronize()
        said = [k for k in eng.launch_kernels(n) if " (in " not in k]
        print(f"[gpu-kernel-names] {dtype} {n}: {said}", flush=True)
        ran = traced(torch, eng, feat, off, out)
        assert [base(k) for k in said] == [base(k) for k in ran], n
        if dtype in ("fp32", "fp8_e4m3"):
            assert [arguments(k) for k in said[:-1]] == [arguments(k) for k in ran[:-1]], n
    i = eng.launch_names().index("enc1.c2")
    for n in sizes:
        assert (eng.launch_kernels(n)[i - 1] == "conv (in enc1.c2)") == (dtype == "bf16" and n == 90), n
    with pytest.raises(ValueError):
        eng.launch_kernels(max(sizes) + 1)
    eng.close()


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp16", "fp8_e4m3"])
def test_track_form_by_batch_size(dtype):
    """The eight-wave track stage up to one event to a compute unit in FP8 (even
    batches past that are faster in the four-wave form) and three to two else."""
    torch = torch_cuda()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    last = cus if dtype == "fp8_e4m3" else 3 * cus // 2
    eng = engine_for(last + 1, dtype)
    for n, waves in ((1, 8), (last, 8), (last + 1, 4)):
        assert eng.launch_kernels(n)[0].endswith(f", {waves}>"), n
    eng.close()
