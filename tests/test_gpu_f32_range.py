"""FP32 convolutions at the top of FP32's range.  Their operands go to the
matrix cores as BF16 pieces, and FP32's largest values (2^128 - 2^119 and
above) round to infinity in BF16, so weights and activations up there, and
infinite activations, must still give what FP32 arithmetic gives: finite
results where the products are finite, infinities of the right sign (here
p = 1) and no NaN where an event overflows."""

import numpy as np
import pytest
import torch

from synth import NetShape, make_events, make_weights, weights_to_blob
from tests import parity, torch_ref
from tests.gpu_util import torch_cuda, run

pytestmark = pytest.mark.gpu

FLT_MAX = np.float32(np.finfo(np.float32).max)


def engine(w, events):
    import paper_2602_19959_amd as pv
    spec = pv.default_spec(max_events=events, max_tracks_total=1500 * events, base_channels=w.shape.base_channels)
    return pv.Engine(weights_to_blob(w), spec)


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("huge", ["activations", "weights"])
def test_largest_finite_operands(width, huge):
    """One value on its way through channel 0 alone, multiplied by up to FLT_MAX
    in every second convolution and by 2^-126 in the others, so that every
    second tensor holds values near FLT_MAX, or every second weight is FLT_MAX.
    Every product is finite."""
    torch_cuda()
    shape = NetShape(base_channels=width)
    w = make_weights(2, shape=shape, zero_bias=True)
    for n, _, _ in shape.tensor_list():
        if not n.startswith("mlp"):
            w[n][:] = 0.0
    w["enc0.c1.b"][0] = 1.0
    order = ["enc0.c2", "enc1.c1", "enc1.c2", "enc2.c1", "enc2.c2", "enc3.c1", "enc3.c2",
             "up2", "dec2.c1", "dec2.c2", "up1", "dec1.c1", "dec1.c2", "up0", "dec0.c1", "dec0.c2"]
    value = 1.0
    for i, n in enumerate(order):
        if (i % 2 == 0) == (huge == "activations"):
            v = FLT_MAX if huge == "weights" or i == 0 else np.float32(FLT_MAX / 4)
        else:
            v = np.float32(2.0 ** -126)
        t = w[n + ".w"]
        if n.startswith("up"):
            t[0, 0, :] = v
        elif n.startswith("dec") and n.endswith("c1"):
            t[0, shape.channels(int(n[3])), 2] = v       # the upsampled half
        else:
            t[0, 0, 2] = v
        value = float(np.float32(value * float(v)))
        assert 0 < value < np.inf
    w["head.w"][0, 0] = np.float32(0.7 / value)
    batch = make_events(2, seed=3)
    eng = engine(w, 2)
    got = run(eng, batch)["prob"]
    if huge == "activations":
        level0 = eng.debug_tensor("enc0.c2", 2).cpu().numpy().reshape(2, width, -1)
        assert np.array_equal(level0[:, 0], np.full_like(level0[:, 0], FLT_MAX))
    eng.close()
    ref = torch.sigmoid(torch_ref.unet(np.zeros(4000), w)).numpy()
    assert 0.6 < ref.min() and ref.max() < 0.7
    for e in range(2):
        assert parity.max_rel(got[e], ref) <= parity.P_REL


def test_overflowing_event_saturates():
    """All weights positive and enc0.c1's near FLT_MAX: positions near a track
    overflow and everything they reach is +infinity, p = 1; no value is NaN and
    the other positions keep their finite p."""
    torch_cuda()
    shape = NetShape()
    w = make_weights(4, shape=shape)
    for n, _, _ in shape.tensor_list():
        if not n.startswith("mlp"):
            w[n][:] = np.abs(w[n]) * np.float32(0.05)
    w["enc0.c1.w"][:] = np.float32(3e38)
    w["head.b"][:] = -1.0
    batch = make_events(3, seed=6)
    eng = engine(w, 3)
    out = run(eng, batch)
    hist = eng.debug_tensor("hist", 3).cpu().numpy().reshape(3, 4000)
    enc = eng.debug_tensor("enc0.c2", 3).cpu().numpy().reshape(3, 32, 4000)
    eng.close()
    assert not np.isnan(enc).any() and (enc == np.inf).any() and np.isfinite(enc).any()
    assert not np.isnan(out["prob"]).any()
    for e in range(3):
        ref = torch.sigmoid(torch_ref.unet(hist[e], w)).numpy()      # FP64 does not overflow: 1 to rounding there
        assert (ref > 1 - 1e-12).any() and (ref < 0.999).any()
        assert parity.max_rel(out["prob"][e], ref) <= parity.P_REL
