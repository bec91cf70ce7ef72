"""Small batches run smaller tiles than full ones: over the sizes where the
choice changes, every output has the bits that the full-batch tiles give (set
explicitly, which pins them), and setting the variants back changes nothing."""

import numpy as np
import pytest

from synth import NetShape, make_events
from tests.gpu_util import torch_cuda, engine_for, make_engine, run, fp8_calibration

pytestmark = pytest.mark.gpu

KEYS = ("prob", "z", "integral", "n_vertices", "bin", "status")


def check(eng, most, sizes):
    batch = make_events(most, seed=13, mix="lognormal")
    small = {}
    for e in sizes:
        print(f"[gpu-batch-tiles] {e} events", flush=True)
        small[e] = run(eng, batch.subset(range(e)))
    base = eng.variants()
    for i, v in enumerate(base):
        if v >= 0:
            assert eng.set_variant(i, v)
    for e in sizes:
        full = run(eng, batch.subset(range(e)))
        for k in KEYS:
            if k in ("z", "integral", "bin"):
                for ev in range(e):
                    n = int(full["n_vertices"][ev])
                    assert np.array_equal(full[k][ev, :n], small[e][k][ev, :n]), (e, k)
            else:
                assert np.array_equal(full[k], small[e][k]), (e, k)
    eng.close()


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp16", "fp8_e4m3"])
def test_small_batch_tiles_give_the_same_bits(dtype):
    torch_cuda()
    check(engine_for(40, dtype), 40, [1, 4, 7, 9, 17, 25, 40])


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8_e4m3"])
def test_small_batch_tiles_wide_network(dtype):
    """64 channels: other column counts, the 64-column head and enc0.c2."""
    torch_cuda()
    shape = NetShape(base_channels=64)
    amax = fp8_calibration(32, 5, shape) if dtype == "fp8_e4m3" else None
    check(make_engine(20, fp8_amax=amax, shape=shape, compute_dtype=dtype), 20, [1, 3, 6, 20])


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp8_e4m3"])
def test_small_batch_tiles_interval_layout(dtype):
    """Short sequences (29 to 104 rows), many to a tile."""
    torch_cuda()
    shape = NetShape(n_levels=3)
    amax = fp8_calibration(32, 5, shape) if dtype == "fp8_e4m3" else None
    check(make_engine(12, fp8_amax=amax, shape=shape, compute_dtype=dtype, unet_layout="interval"), 12, [1, 2, 12])


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp16", "fp8_e4m3"])
@pytest.mark.parametrize("boundary", [0.0, 2.5])
def test_track_and_peak_forms_give_the_same_bits(dtype, boundary):
    """Few events spread each event over more waves (track stage: 1 to 128, to
    384, more; peaks: to 256, more).  Heavy-tailed events of one to six chunks,
    the smallest of 5 tracks, without and with boundary tracks, at another half
    window than the default's."""
    torch_cuda()
    most = 390
    batch = make_events(most, seed=17, mix="lognormal")
    eng = engine_for(most, dtype, boundary_mm=boundary, half_window=5 if boundary else 3)
    full = run(eng, batch)
    for n in (1, 128, 129, 257, 384):
        print(f"[gpu-batch-tiles] {dtype} {n} events, boundary {boundary}", flush=True)
        part = run(eng, batch.subset(range(n)))
        for k in ("prob", "status", "n_vertices"):
            assert np.array_equal(part[k], full[k][:n]), (n, k)
        for e in range(n):
            v = int(full["n_vertices"][e])
            for k in ("z", "integral", "bin", "peak_prob"):
                assert np.array_equal(part[k][e, :v], full[k][e, :v]), (n, e, k)
    eng.close()
