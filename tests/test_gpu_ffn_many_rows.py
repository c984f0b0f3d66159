"""Feed-forward calls of millions of rows, whose tile indices leave the range of a 32-bit
reciprocal product or whose outputs pass 4 GiB: every row against the same rows run in parts, and rows spread over the
call (the last ones among them) against the CPU oracle.  The module works row by row."""

import numpy as np
import pytest

from oracle import core
from workloads import make_ffn

pytestmark = pytest.mark.gpu


# rows of 64 -> 256 channels in more than 2^16 token tiles; an output of more than 2^32 bytes
@pytest.mark.parametrize("rows,d,d_ff", [(4692372, 64, 256), (4200001, 1024, 64)])
def test_many_rows(gpu_lib, rows, d, d_ff):
    import torch

    print(f"[many rows] rows={rows} d={d} d_ff={d_ff}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(rows)
    z = torch.empty((rows, d), dtype=torch.int8, device="cuda").random_(-127, 128, generator=gen)
    f = make_ffn(d, "calibrated", seed=3, S_z=1.0 / 32, d_ff=d_ff)
    mod = gpu_lib.FeedForward(f, max_rows=rows)
    out = mod(z)
    part = 1 << 18
    for r in range(0, rows, part):
        assert torch.equal(out[r:r + part], mod(z[r:r + part])), r
    at = np.unique(np.concatenate([np.linspace(0, rows - 1, 300).astype(np.int64), np.arange(rows - 130, rows)]))
    sel = torch.from_numpy(at).cuda()
    assert np.array_equal(out[sel].cpu().numpy(), core.ffn_module(f, z[sel].cpu().numpy()))
    mod.close()
