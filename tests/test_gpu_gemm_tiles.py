"""Every tile shape of the projection GEMMs at its edges: token counts one off a tile, a
single token, channel counts that leave the last tile mostly empty, contraction lengths
of one step and of odd multiples of 64, in each of the three epilogues (Swish and residual
through the feed-forward module, plain through the convolution module, the Q|K|V and
position layouts through the block), against the CPU oracle, byte for byte.

The sizes are chosen so that the launch picks, in order, the 128 x 32, 64 x 64, 128 x 64,
256 x 64 and 256 x 128 shapes for at least one product of the case.
"""

import numpy as np
import pytest

from oracle import core
from workloads import make_block, make_conv, make_ffn
from workloads.generate import ConfigShape

pytestmark = pytest.mark.gpu


def _rows(rng, rows, d):
    return np.clip(np.rint(rng.normal(0.0, 32.0, size=(rows, d))), -127, 127).astype(np.int8)


@pytest.mark.parametrize("rows,d,d_ff", [
    (1, 64, 64), (31, 64, 192), (33, 192, 320), (1025, 192, 1024), (513, 1024, 448), (2049, 320, 1600),
    (2047, 1024, 4096), (6401, 256, 1024), (8193, 1024, 1024)])
def test_feed_forward(gpu_lib, rows, d, d_ff):
    import torch

    print(f"[tiles] ffn rows={rows} d={d} d_ff={d_ff}", flush=True)
    rng = np.random.default_rng(rows * 7 + d)
    z = _rows(rng, rows, d)
    f = make_ffn(d, "calibrated", seed=rows + d_ff, S_z=1.0 / 32, d_ff=d_ff)
    mod = gpu_lib.FeedForward(f, max_rows=rows)
    out = mod(torch.from_numpy(z).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), core.ffn_module(f, z))
    mod.close()


@pytest.mark.parametrize("B,T,d", [(1, 1, 64), (1, 33, 192), (3, 65, 320), (2, 1025, 256), (5, 821, 1024)])
def test_convolution(gpu_lib, B, T, d):
    import torch

    print(f"[tiles] conv B={B} T={T} d={d}", flush=True)
    rng = np.random.default_rng(B * T + d)
    z = _rows(rng, B * T, d).reshape(B, T, d)
    lengths = rng.integers(1, T + 1, size=B).astype(np.int32)
    cv = make_conv(d, "calibrated", seed=T + d, S_z=1.0 / 32)
    mod = gpu_lib.ConvModule(cv, max_batch=B, max_T=T)
    out = mod(torch.from_numpy(z).cuda(), lengths=lengths)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), core.conv_module(cv, z, lengths=lengths))
    mod.close()


# V^T is written in whole 64-key blocks by every shape, the position table at its own row
# offset: T on either side of a block, and enough utterances to reach the large shapes
@pytest.mark.parametrize("B,T,d,H", [(1, 1, 64, 1), (1, 63, 128, 1), (2, 65, 320, 5), (9, 129, 512, 4), (33, 127, 1024, 8),
                                     (13, 257, 1024, 16)])
def test_projections(gpu_lib, B, T, d, H):
    import torch

    print(f"[tiles] block B={B} T={T} d={d} H={H}", flush=True)
    rng = np.random.default_rng(B + T + d)
    lengths = rng.integers(1, T + 1, size=B)
    blk = make_block(ConfigShape("tiles", B=B, T=T, d_model=d, n_heads=H), T, rng, "calibrated", lengths=lengths)
    mod = gpu_lib.RelPosAttn.from_block(blk)
    y = mod(torch.from_numpy(blk.x).cuda(), torch.from_numpy(blk.pos_table).cuda(), lengths=blk.lengths)
    inter = {k: mod.intermediate(i, (B, T, d) if k != "p" else (2 * T - 1, d))
             for k, i in (("q", 0), ("k", 1), ("v", 2), ("p", 3))}
    torch.cuda.synchronize()
    ref, tr = core.relpos_attn(blk, trace=True)
    for k, t in inter.items():
        assert np.array_equal(t.cpu().numpy(), tr[k]), k
    assert np.array_equal(y.cpu().numpy(), ref)
    mod.close()
