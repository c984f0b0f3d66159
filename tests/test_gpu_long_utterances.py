"""Utterances past the length whose score rows fit on chip (3968 frames), where a workgroup
passes part of its scores through memory: one frame past the limit, one and two spilled
parts at their edges, ragged batches whose shorter utterances need no part or no work at
all, both head widths, both score forms, the kept position projection and the
no-allocation run, against the CPU oracle."""

import numpy as np
import pytest
from oracle import core
from workloads import make_block
from workloads.generate import ConfigShape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,H,lengths", [
    (3968, 64, 1, [3968]), (3969, 64, 1, [3969]), (4032, 128, 1, [4032, 3967]), (4033, 128, 2, [4033, 17, 3969]),
    (7936, 64, 1, [7936]), (7937, 64, 1, [7937]), (8000, 128, 1, [8000, 1]), (6001, 128, 2, [4100, 6001])])
def test_long(gpu_lib, T, d, H, lengths):
    import torch

    ipk = gpu_lib
    B = len(lengths)
    print(f"[long] T={T} d={d} H={H} lengths={lengths}", flush=True)
    rng = np.random.default_rng(T + d)
    blk = make_block(ConfigShape("long", B=B, T=T, d_model=d, n_heads=H), T, rng, "calibrated", lengths=lengths)
    x, pe = torch.from_numpy(blk.x).cuda(), torch.from_numpy(blk.pos_table).cuda()
    mod = ipk.RelPosAttn.from_block(blk)
    ref = core.relpos_attn(blk)
    runs = {"run": lambda: mod(x, pe, lengths=blk.lengths)}

    def wide():
        ipk.ipk_relpos_attn_set_score_path(mod.handle, ipk.IPK_SCORE_WIDE)
        y = mod(x, pe, lengths=blk.lengths)
        ipk.ipk_relpos_attn_set_score_path(mod.handle, ipk.IPK_SCORE_AUTO)
        return y

    def kept():
        mod.cache_positions(pe)
        return mod(x, None, lengths=blk.lengths)

    runs["64-bit scores"] = wide
    runs["kept positions"] = kept
    runs["no allocation"] = lambda: mod.run_noalloc(x, pe, lengths=blk.lengths, y=torch.empty_like(x))
    for name, run in runs.items():
        y = run()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), ref), name
    mod.close()


def test_limit(gpu_lib):
    rng = np.random.default_rng(1)
    blk = make_block(ConfigShape("long", B=1, T=64, d_model=64, n_heads=1), 64, rng, "calibrated")
    with pytest.raises(gpu_lib.IpkError) as e:
        gpu_lib.RelPosAttn.from_block(blk, max_T=8001)
    assert e.value.status == gpu_lib.IPK_ERR_UNSUPPORTED
