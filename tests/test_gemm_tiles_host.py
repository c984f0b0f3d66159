"""Index arithmetic of the projection GEMMs on the host (no GPU): the division by launch-time
divisors, and the tile decomposition of every product that the entry points accept, at
their largest sizes and in every tile shape.  A quotient one off would send a tile's
loads and stores outside its operands."""

import numpy as np
import pytest

import host_plans

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
