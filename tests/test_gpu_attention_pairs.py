"""The attention core in batches of short utterances, where two workgroups may share a CU:
paired 64-query (four key splits) and 32-query (eight) workgroups, at d_k 128 in the kernel
compiled for half the registers and at d_k 64 in the ordinary one, from one 64-key chunk to
many, the longest utterance of which two 64-query ones fit (704 frames) and one past it, and
the unpaired plans around them; ragged lengths and both score forms, against the CPU
oracle.  The plan of each case is asserted on the CPU, by test_attention_plan_host.py."""

import numpy as np
import pytest

from oracle import core
from workloads import make_block
from workloads.generate import ConfigShape

pytestmark = pytest.mark.gpu


CASES = [(34, 33, 1024, 8), (40, 130, 256, 2), (11, 375, 1024, 8), (64, 61, 512, 8), (30, 640, 256, 2), (30, 641, 256, 2),
         (9, 1030, 256, 2), (80, 80, 256, 2), (12, 1020, 256, 2), (10, 1216, 256, 2), (40, 300, 256, 2),
         (18, 704, 256, 2), (18, 705, 256, 2), (80, 80, 256, 4), (40, 300, 256, 4)]


@pytest.mark.parametrize("B,T,d,H", CASES)
def test_pairs(gpu_lib, B, T, d, H):
    import torch

    ipk = gpu_lib
    print(f"[pairs] B={B} T={T} d={d} H={H}", flush=True)
    rng = np.random.default_rng(B + T + d)
    lengths = rng.integers(1, T + 1, size=B)
    lengths[:3] = [T, 1, max(1, T // 2)]
    blk = make_block(ConfigShape("pairs", B=B, T=T, d_model=d, n_heads=H), T, rng, "calibrated", lengths=lengths)
    mod = ipk.RelPosAttn.from_block(blk)
    x, pe = torch.from_numpy(blk.x).cuda(), torch.from_numpy(blk.pos_table).cuda()
    ref = core.relpos_attn(blk)
    for path in (ipk.IPK_SCORE_AUTO, ipk.IPK_SCORE_WIDE):
        ipk.ipk_relpos_attn_set_score_path(mod.handle, path)
        y = mod(x, pe, lengths=blk.lengths)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), ref), path
    mod.close()
