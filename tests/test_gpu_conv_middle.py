"""The convolution module's middle kernel (GLU, depthwise taps, INT16 BatchNorm, Swish) at
the edges of its tiles: frame counts around a frame quad and around the largest tile,
channel counts that leave lanes idle, launches of several tiles per workgroup, utterances
that end inside a quad, and requantization constants that saturate (the accumulator
bound) or vanish, against the CPU oracle."""

import numpy as np
import pytest

from oracle import core
from workloads import make_conv

pytestmark = pytest.mark.gpu


def _check(ipk, cv, B, T, seed):
    import torch

    d = cv.d_model
    rng = np.random.default_rng(seed)
    z = np.clip(np.rint(rng.normal(0.0, 32.0, size=(B, T, d))), -127, 127).astype(np.int8)
    lengths = rng.integers(1, T + 1, size=B).astype(np.int32)
    lengths[0] = T
    mod = ipk.ConvModule(cv, max_batch=B, max_T=T)
    out = mod(torch.from_numpy(z).cuda(), lengths=lengths)
    o = mod.intermediate(ipk.IPK_CONV_O, B, T)
    v = mod.intermediate(ipk.IPK_CONV_V, B, T)
    torch.cuda.synchronize()
    ref, tr = core.conv_module(cv, z, lengths=lengths, trace=True)
    assert np.array_equal(v.cpu().numpy(), tr["v"])
    assert np.array_equal(o.cpu().numpy(), tr["o"])
    assert np.array_equal(out.cpu().numpy(), ref)
    mod.close()


@pytest.mark.parametrize("regime", ["literal", "calibrated"])
@pytest.mark.parametrize("B,T,d", [(1, 1, 64), (1, 3, 320), (2, 5, 256), (3, 56, 192), (2, 57, 576), (70, 61, 64), (31, 375, 320),
                                   (5, 1021, 512)])
def test_middle(gpu_lib, B, T, d, regime):
    print(f"[conv middle] B={B} T={T} d={d} {regime}", flush=True)
    _check(gpu_lib, make_conv(d, regime, seed=B + T + d, S_z=1.0 / 32), B, T, seed=T)


@pytest.mark.parametrize("shift", [1, 16, 31, 32, 40])
def test_requantization_range(gpu_lib, shift):
    """Multipliers from 0 to 2^23 - 1 and biases up to the limit, at every kind of shift."""
    print(f"[conv middle] shift_dw={shift}", flush=True)
    d = 256
    cv = make_conv(d, "calibrated", seed=shift, S_z=1.0 / 32)
    rng = np.random.default_rng(shift)
    cv.shift_dw = shift
    cv.mult_dw = (rng.integers(0, 1 << 23, size=d) >> rng.integers(0, 23, size=d)).astype(np.int32)
    cv.mult_dw[:4] = [0, 1, (1 << 23) - 1, (1 << 23) - 1]
    cv.bias_dw = (rng.integers(-(1 << 30) + 1, 1 << 30, size=d) >> rng.integers(0, 30, size=d)).astype(np.int32)
    cv.bias_dw[:4] = [(1 << 30) - 1, -(1 << 30) + 1, (1 << 30) - 1, -(1 << 30) + 1]
    _check(gpu_lib, cv, 2, 70, seed=shift)
