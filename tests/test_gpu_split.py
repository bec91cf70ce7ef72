"""The FP32 convolutions' tiles (FP32 operands as three BF16 pieces each) at
the sizes where a tile can go wrong: batches whose rows end inside, at and just
past a tile, a single short event, the shortest sequences, one 32-channel chunk
and many.  Every tile variant must give the default's bits, p must be within the
FP32 bar of the oracle (tests/parity.py), and an event's bits must not depend on
the batch."""

import numpy as np
import pytest

import oracle
from synth import NetShape, make_events
from tests import parity
from tests.gpu_util import torch_cuda, make_engine, run, geometry, weights

pytestmark = pytest.mark.gpu


# (bins, bins per interval, levels, width, events): level-0 rows are events x (bins + 4)
@pytest.mark.parametrize("n_bins,bpi,levels,width,events", [
    (60, 20, 2, 32, 1),          # 64 rows: half of the smallest tile of 128
    (124, 31, 2, 32, 1),         # 128 rows: one tile exactly
    (128, 32, 2, 32, 2),         # 264 rows: 8 past two tiles of 128, one of 256
    (508, 127, 2, 64, 1),        # 512 rows, 64 columns in the head
    (512, 128, 6, 32, 3),        # six levels: 16 positions and 1024 channels at the bottom
    (4000, 100, 4, 64, 1),
])
def test_split_tiles(n_bins, bpi, levels, width, events):
    torch_cuda()
    shape = NetShape(n_out=bpi, n_levels=levels, base_channels=width)
    eng = make_engine(events, shape=shape, n_bins=n_bins, bins_per_interval=bpi, max_peaks_per_event=n_bins // 2)
    batch = make_events(events, seed=11)
    print(f"[gpu-split] {n_bins} bins, {levels} levels, width {width}, {events} events", flush=True)
    out = run(eng, batch)
    geo = geometry(eng)
    refs = oracle.run_batch(batch, weights(0, shape), geo)
    for e in range(events):
        assert parity.max_rel(out["prob"][e], refs[e]["p"]) <= parity.P_REL, e
    parity.exact_peaks_all(out, geo)
    base = eng.variants()
    for v in range(eng.variant_count(2)):
        if not [i for i in range(len(base)) if base[i] >= 0 and eng.set_variant(i, v)]:
            continue
        assert np.array_equal(run(eng, batch)["prob"], out["prob"]), v
        for i in range(len(base)):
            if base[i] >= 0:
                eng.set_variant(i, base[i])
    if events > 1:
        last = run(eng, batch.subset([events - 1]))
        assert np.array_equal(last["prob"][0], out["prob"][events - 1])
    eng.close()
