"""Launch planning of the projection GEMMs on the host (no GPU): the division by launch-time
divisors, and the tile decomposition of every product that the entry points accept, at
their largest sizes and in every tile shape (a quotient one off would send a tile's
loads and stores outside its operands); and that the GPU test of the tile shapes does run
each shape, with a remainder, in each epilogue and layout."""

import numpy as np
import pytest

import host_plans
from host_plans import PLAIN, RESID, SWISH, gemm_shape
from tests import test_gpu_gemm_tiles as gpu

SHAPES = [(256, 256), (256, 128), (256, 64), (128, 64), (64, 64), (128, 32)]  # channels x tokens
ROW_LIMIT = 2 ** 31 - 1  # of max_rows d_ff (feed-forward) and max_batch max_T 2 d_model (convolution)


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return host_plans.load(str(tmp_path_factory.mktemp("host_plans")))


def test_division_is_exact_below_2_31(plans):
    rng = np.random.default_rng(1)
    ds = {1, 2, 3, 5, 7, 64, 65, 2 ** 30 - 1, 2 ** 30, 2 ** 30 + 1, 2 ** 31 - 1} | {
        int(v) for v in np.exp2(rng.uniform(0, 31, size=3000))}
    for d in sorted(ds):
        q = np.unique(rng.integers(0, (2 ** 31 - 1) // d + 1, size=2000, dtype=np.int64))
        xs = np.concatenate([q * d + k for k in (-1, 0, 1)] + [rng.integers(0, 2 ** 31, size=500, dtype=np.int64),
                                                               np.array([0, 1, 2 ** 31 - 2, 2 ** 31 - 1])])
        xs = np.ascontiguousarray(xs[(xs >= 0) & (xs < 2 ** 31)], dtype=np.uint32)
        assert plans.div_fault(d, xs.ctypes.data, xs.size) == -1, d


# row-major products: feed-forward calls at the accepted row limit and at the row count of a
# wrong quotient, widths that a limit of 2^32 on x d would refuse
@pytest.mark.parametrize("d,d_ff,rows", [(64, 256, 4692372)] + [
    (d, f, ROW_LIMIT // f) for d in (64, 256, 1024, 4096) for f in (64, 128, 192, 256, 320, 448, 512, 1024, 4096)])
def test_feed_forward_tiles(plans, d, d_ff, rows):
    for n in {d, d_ff}:
        for tn, tm in SHAPES:
            assert plans.tile_grid_fault(1, rows, n, tn, tm) == 0, (n, tn, tm)


# Q|K|V, the position table, the output projection and the convolution's products at the
# largest batch and length
@pytest.mark.parametrize("d", [64, 320, 1024, 4096, 16384])
@pytest.mark.parametrize("B,T", [(256, 8000), (128, 8000), (256, 3967), (1, 8000), (1, 1)])
def test_block_and_convolution_tiles(plans, d, B, T):
    for tn, tm in SHAPES[:5]:
        if tn * tm >= 128 * 64 or B * T < 2 ** 18:
            assert plans.tile_grid_fault(B, T, 3 * d, tn, tm) == 0, (tn, tm)
            assert plans.tile_grid_fault(1, B * T, d, tn, tm) == 0, (tn, tm)
        assert plans.tile_grid_fault(1, 2 * T - 1, d, tn, tm) == 0, (tn, tm)


# what the products of the GPU test's cases take: W1 and W2; PW1 and PW2; Q|K|V with the
# position table, the output projection and the position table alone
FFN = {(8193, 64, 64): ((64, 64), (64, 64)), (3589, 576, 832): ((256, 64), (256, 64)),
       (12375, 448, 448): ((256, 128), (256, 128)), (14577, 960, 192): ((256, 64), (256, 256)),
       (8804, 128, 1600): ((256, 256), (128, 64)), (12305, 1024, 1024): ((256, 256), (256, 256)),
       (4113, 1024, 4096): ((256, 64), (256, 128)), (1223, 64, 832): ((128, 64), (128, 32)),
       (1232, 832, 64): ((128, 32), (128, 64))}
CONV = {(7, 881, 1024): ((256, 256), (256, 128)), (4, 2723, 576): ((256, 256), (128, 64)),
        (5, 1961, 320): ((256, 128), (128, 64)), (11, 227, 832): ((128, 64), (256, 64)),
        (3, 4097, 448): ((128, 64), (256, 128))}
BLOCK = {(33, 16, 192, 3): ((128, 64), (128, 32), (128, 32)), (33, 65, 576, 9): ((256, 128), (128, 64), (128, 32)),
         (33, 193, 576, 9): ((256, 256), (128, 64), (128, 32)), (33, 200, 320, 5): ((128, 64), (256, 64), (128, 32)),
         (33, 752, 192, 3): ((128, 64), (256, 128), (128, 32)), (1, 899, 576, 9): ((256, 64), (128, 32), (128, 64)),
         (1, 1253, 832, 13): ((128, 64), (128, 64), (256, 64)), (33, 272, 64, 1): ((64, 64), (64, 64), (128, 32))}
POSITION = {(8000, 64, 1): (64, 64), (8000, 512, 4): (256, 128), (8000, 1024, 8): (256, 256)}


def test_the_gpu_cases_take_these_shapes(plans):
    assert list(FFN) == gpu.FFN_SHAPES and list(CONV) == gpu.CONV_SHAPES and list(BLOCK) == gpu.BLOCK_SHAPES
    for (rows, d, f), (up, down) in FFN.items():
        assert gemm_shape(plans, [(1, rows, f)], d, SWISH) == up, (rows, d, f)
        assert gemm_shape(plans, [(1, rows, d)], f, RESID) == down, (rows, d, f)
    for (B, T, d), (pw1, pw2) in CONV.items():
        assert gemm_shape(plans, [(1, B * T, 2 * d)], d, PLAIN) == pw1, (B, T, d)
        assert gemm_shape(plans, [(1, B * T, d)], d, RESID) == pw2, (B, T, d)
    for (B, T, d, H), (qkv, out, pos) in BLOCK.items():
        assert gemm_shape(plans, [(B, T, 3 * d), (1, 2 * T - 1, d)], d, PLAIN, min_tm=64) == qkv, (B, T, d)
        assert gemm_shape(plans, [(1, B * T, d)], d, PLAIN) == out, (B, T, d)
        assert gemm_shape(plans, [(1, 2 * T - 1, d)], d, PLAIN) == pos, (B, T, d)
    assert list(POSITION) == gpu.POSITION_SHAPES
    for (T, d, H), pos in POSITION.items():
        assert gemm_shape(plans, [(1, 2 * T - 1, d)], d, PLAIN) == pos, (T, d)


def _marked(test):
    """The parameter sets of one of the GPU test's parametrised functions."""
    return [m.args[1] for m in test.pytestmark if m.name == "parametrize" and "wide" not in m.args[0]][0]


def test_every_shape_runs_with_a_remainder_in_every_epilogue(plans):
    seen = {k: set() for k in ("swish", "residual", "row-major plain", "Q|K|V", "position")}

    def add(kind, products, K, epilogue, min_tm=32):
        tn, tm = gemm_shape(plans, products, K, epilogue, min_tm)
        nb, rows, N = products[0]
        if rows % tm and (N % tn or tn == 64):  # channels come in multiples of 64
            seen[kind].add((tn, tm))

    for rows, d, f in _marked(gpu.test_feed_forward) + gpu.FFN_SHAPES:
        add("swish", [(1, rows, f)], d, SWISH)
        add("residual", [(1, rows, d)], f, RESID)
    for B, T, d in _marked(gpu.test_convolution) + gpu.CONV_SHAPES:
        add("row-major plain", [(1, B * T, 2 * d)], d, PLAIN)
        add("residual", [(1, B * T, d)], d, RESID)
    for B, T, d, H in _marked(gpu.test_projections) + gpu.BLOCK_SHAPES:
        add("Q|K|V", [(B, T, 3 * d), (1, 2 * T - 1, d)], d, PLAIN, 64)
        add("row-major plain", [(1, B * T, d)], d, PLAIN)
    for T, d in [(T, d) for _, T, d, _ in gpu.BLOCK_SHAPES] + [(T, d) for T, d, _ in gpu.POSITION_SHAPES]:
        seen["position"].add(gemm_shape(plans, [(1, 2 * T - 1, d)], d, PLAIN))  # 2 T - 1 is no multiple of a tile
    every = set(SHAPES)
    assert seen["Q|K|V"] == every - {(128, 32)}  # V^T is written in blocks of 64 keys
    for kind in ("swish", "residual", "row-major plain", "position"):
        assert seen[kind] == every, (kind, every - seen[kind])
