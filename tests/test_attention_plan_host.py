"""Which workgroup shapes the attention core takes for the cases of its GPU tests (no GPU):
the launch's own plan, so that a refitted constant cannot silently move a case to another
kernel than the one it is there for."""

import pytest

import host_plans
from tests import test_gpu_attention_pairs as pairs

Q64, Q48, Q32 = (4, 2), (8, 3), (8, 2)  # 64-, 48- and 32-query workgroups


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return host_plans.load(str(tmp_path_factory.mktemp("host_plans")))


PAIRS = {(34, 33, 1024, 8): (Q64, None, True), (40, 130, 256, 2): (Q48, None, False),
         (11, 375, 1024, 8): (Q48, None, False), (64, 61, 512, 8): (Q64, None, True),
         (30, 640, 256, 2): (Q48, Q32, False), (30, 641, 256, 2): (Q48, Q32, False), (9, 1030, 256, 2): (Q48, Q32, False),
         (80, 80, 256, 2): (Q32, None, True), (12, 1020, 256, 2): (Q32, None, True), (10, 1216, 256, 2): (Q32, None, True),
         (40, 300, 256, 2): (Q64, None, True), (18, 704, 256, 2): (Q64, None, True), (18, 705, 256, 2): None,
         (80, 80, 256, 4): (Q32, None, True), (40, 300, 256, 4): (Q64, None, True)}


def test_pair_cases(plans):
    assert list(PAIRS) == pairs.CASES
    for (B, T, d, H), want in PAIRS.items():
        got = host_plans.attn_shape(plans, B, T, d, H)
        if want is None:  # past the length of which two 64-query workgroups fit
            assert not got[2], (B, T, d, H)
        else:
            assert got == want, (B, T, d, H)


def test_two_64_query_workgroups_fit_up_to_704_frames(plans):
    shapes = {T: {host_plans.attn_shape(plans, B, T, 256, 2) for B in range(1, 129)} for T in (704, 705)}
    assert any(p and s == Q64 for s, _, p in shapes[704]) and not any(p and s == Q64 for s, _, p in shapes[705])


@pytest.mark.parametrize("d,H", [(64, 1), (128, 1), (1024, 8), (1024, 16)])
def test_spilling_workgroups_past_3968_frames(plans, d, H):
    for B in (1, 2, 16, 256):
        assert host_plans.attn_shape(plans, B, 3968, d, H)[0] is not None
        for T in (3969, 4500, 8000):
            assert host_plans.attn_shape(plans, B, T, d, H) == (None, None, False)
