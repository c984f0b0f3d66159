"""The integer LayerNorm kernel over its row layouts (16, 32 or 64 lanes per row, one or
four rows per lane, several pieces per lane), both forms of the final shift (below 32 and
from 32 on) and both ranges of sigma (at most 256, above), against the CPU oracle."""

import types

import numpy as np
import pytest

from oracle import core

pytestmark = pytest.mark.gpu

# d on either side of each layout's limit; the large row counts reach four rows per lane,
# with a remainder
SHAPES = [(1, 16), (8195, 16), (7, 256), (8197, 256), (33, 272), (4099, 512), (5, 528), (2051, 1024), (9, 1040), (3, 2064),
          (2, 4112), (2, 8208), (2, 16384)]


@pytest.mark.parametrize("ln_shift", [20, 31, 32, 40])
@pytest.mark.parametrize("rows,d", SHAPES)
def test_layernorm(gpu_lib, rows, d, ln_shift):
    import torch

    print(f"[layernorm] rows={rows} d={d} shift={ln_shift}", flush=True)
    rng = np.random.default_rng(rows + d + ln_shift)
    z = rng.integers(-128, 128, size=(rows, d)).astype(np.int8)
    # rows of small spread (sigma of at most 256, down to the constant row's 1) among the wide ones
    for r in range(0, rows, 3):
        z[r] = np.clip(rng.integers(-100, 100) + rng.integers(-1, 2, size=d) * (r % 2), -128, 127)
    p = types.SimpleNamespace(
        ln_mult=rng.integers(-(1 << 24) + 1, 1 << 24, size=d).astype(np.int32) >> max(0, 36 - ln_shift) // 2,
        ln_bias=rng.integers(-(1 << (ln_shift + 6)), 1 << (ln_shift + 6), size=d), ln_shift=ln_shift)
    p.ln_bias[0], p.ln_bias[d - 1] = (1 << 56) - 1, -(1 << 56) + 1
    m = gpu_lib.LayerNorm(d, p)
    x = m(torch.from_numpy(z).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(x.cpu().numpy(), core.layernorm(z, p))
    m.close()
