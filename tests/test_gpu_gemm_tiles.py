"""Every tile shape of the projection GEMMs at its edges: token counts one off a tile, a
single token, channel counts that leave the last tile mostly empty, contraction lengths
of one step and of odd multiples of 64, in each of the three epilogues (Swish and residual
through the feed-forward module, plain through the convolution module and the output
projection, the Q|K|V and position layouts through the block), against the CPU oracle, byte
for byte; and in both forms of Eq. 7 and of the residual add (the wide cases take the
64-bit ones in every product).

Which shape each product of each case takes is asserted on the CPU, by
test_gemm_tiles_host.py, from the launch's own rule.
"""

import dataclasses

import numpy as np
import pytest

from oracle import core
from tests.test_gpu_requant_forms import _deeper_shift
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


# the larger shapes with a remainder of rows and of channels, and the widths that take them;
# wide: shifts above 16, and residual multipliers past the 32-bit form
FFN_SHAPES = [(8193, 64, 64), (3589, 576, 832), (12375, 448, 448), (14577, 960, 192), (8804, 128, 1600),
              (12305, 1024, 1024), (4113, 1024, 4096), (1223, 64, 832), (1232, 832, 64)]
CONV_SHAPES = [(7, 881, 1024), (4, 2723, 576), (5, 1961, 320), (11, 227, 832), (3, 4097, 448)]
BLOCK_SHAPES = [(33, 16, 192, 3), (33, 65, 576, 9), (33, 193, 576, 9), (33, 200, 320, 5), (33, 752, 192, 3),
                (1, 899, 576, 9), (1, 1253, 832, 13), (33, 272, 64, 1)]
POSITION_SHAPES = [(8000, 64, 1), (8000, 512, 4), (8000, 1024, 8)]  # T, d, H


def _wide(p, *names):
    """``p`` with the Eq. 7 constants mult<name>, shift<name> at shifts above 16 and the residual's multipliers at their limit."""
    new = {"m_z": (1 << 23) - 1, "m_y": (1 << 23) - 1, "shift_r": 24}
    for n in names:
        new["mult" + n], new["shift" + n] = _deeper_shift(getattr(p, "mult" + n), getattr(p, "shift" + n), 3)
        assert new["shift" + n] > 16
    return dataclasses.replace(p, **new)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("rows,d,d_ff", FFN_SHAPES)
def test_feed_forward_shapes(gpu_lib, rows, d, d_ff, wide):
    import torch

    print(f"[tiles] ffn rows={rows} d={d} d_ff={d_ff} wide={wide}", flush=True)
    z = _rows(np.random.default_rng(rows + d), rows, d)
    f = make_ffn(d, "calibrated", seed=rows, S_z=1.0 / 32, d_ff=d_ff)
    f = _wide(f, "1", "2") if wide else f
    mod = gpu_lib.FeedForward(f, max_rows=rows)
    out = mod(torch.from_numpy(z).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), core.ffn_module(f, z))
    mod.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("B,T,d", CONV_SHAPES)
def test_convolution_shapes(gpu_lib, B, T, d, wide):
    import torch

    print(f"[tiles] conv B={B} T={T} d={d} wide={wide}", flush=True)
    rng = np.random.default_rng(B * T + d)
    z = _rows(rng, B * T, d).reshape(B, T, d)
    lengths = rng.integers(1, T + 1, size=B).astype(np.int32)
    cv = make_conv(d, "calibrated", seed=T, S_z=1.0 / 32)
    cv = _wide(cv, "_pw1", "_pw2") if wide else cv
    mod = gpu_lib.ConvModule(cv, max_batch=B, max_T=T)
    out = mod(torch.from_numpy(z).cuda(), lengths=lengths)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), core.conv_module(cv, z, lengths=lengths))
    mod.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("B,T,d,H", BLOCK_SHAPES)
def test_block_shapes(gpu_lib, B, T, d, H, wide):
    import torch

    print(f"[tiles] block B={B} T={T} d={d} H={H} wide={wide}", flush=True)
    rng = np.random.default_rng(B + T + d)
    lengths = rng.integers(1, T + 1, size=B)
    blk = make_block(ConfigShape("tiles", B=B, T=T, d_model=d, n_heads=H), T, rng, "calibrated", lengths=lengths)
    if wide:
        blk.consts = dict(blk.consts)
        for n in ("q", "pos", "out"):  # one matrix of Q|K|V puts the whole stack there
            blk.consts["mult_" + n], blk.consts["shift_" + n] = _deeper_shift(blk.consts["mult_" + n],
                                                                              blk.consts["shift_" + n], 3)
    mod = gpu_lib.RelPosAttn.from_block(blk)
    x, pe = torch.from_numpy(blk.x).cuda(), torch.from_numpy(blk.pos_table).cuda()
    y = mod(x, pe, lengths=blk.lengths)
    inter = {k: mod.intermediate(i, (B, T, d) if k != "p" else (2 * T - 1, d))
             for k, i in (("q", 0), ("k", 1), ("v", 2), ("p", 3))}
    mod.cache_positions(pe)  # the position product alone
    kept = mod(x, None, lengths=blk.lengths)
    inter["p kept"] = mod.intermediate(3, (2 * T - 1, d))
    torch.cuda.synchronize()
    ref, tr = core.relpos_attn(blk, trace=True)
    for k, t in inter.items():
        assert np.array_equal(t.cpu().numpy(), tr[k[0]]), k
    for out in (y, kept):
        assert np.array_equal(out.cpu().numpy(), ref)
    mod.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("T,d,H", POSITION_SHAPES)
def test_position_shapes(gpu_lib, T, d, H, wide):
    import torch

    print(f"[tiles] position table T={T} d={d} wide={wide}", flush=True)
    blk = make_block(ConfigShape("tiles", B=1, T=T, d_model=d, n_heads=H), T, np.random.default_rng(T + d), "calibrated")
    c = blk.consts = dict(blk.consts)
    if wide:
        c["mult_pos"], c["shift_pos"] = _deeper_shift(c["mult_pos"], c["shift_pos"], 3)
    mod = gpu_lib.RelPosAttn.from_block(blk)
    mod.cache_positions(torch.from_numpy(blk.pos_table).cuda())
    mod(torch.from_numpy(blk.x).cuda(), None)
    p = mod.intermediate(3, (2 * T - 1, d))
    torch.cuda.synchronize()
    assert np.array_equal(p.cpu().numpy(), core.linear(blk.pos_table, blk.w_pos, c["mult_pos"], c["shift_pos"]))
    mod.close()
