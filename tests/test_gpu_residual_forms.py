"""Both forms of the residual add z2 = clamp8(RS(m_z z + m_y y, 1, n)) in the GEMM epilogues
against the CPU oracle: 32-bit integers while (m_z + m_y) 128 + 2^(n-1) stays below 2^31
(every workload's multipliers at shift 16, and here shifts up to 30 and the bound itself),
64-bit ones past it and at shifts above 31, up to the largest multipliers and shift, through
the MHSA, feed-forward and convolution modules.  Inputs hold the int8 extremes, -128 too."""

import dataclasses

import numpy as np
import pytest

from oracle import core
from tests.test_gpu_conv import _check as _check_conv
from tests.test_gpu_ffn import _check as _check_ffn
from tests.test_gpu_residual import _check as _check_mhsa
from workloads import make_conv, make_ffn, make_residual, make_workload

TOP = (1 << 23) - 1  # the largest multiplier
AT_BOUND = ((1 << 31) - (1 << 22)) // 128 - 1 - TOP  # with m_z = TOP, n = 23: the last m_y of the 32-bit form

# (m_z, m_y, n, 64-bit form)
FORMS = [(52429, 70000, 17, False), (TOP, 1 << 22, 23, False), (TOP, AT_BOUND, 23, False), (TOP, AT_BOUND + 1, 23, True),
         (TOP, 4000000, 30, False), (0, TOP, 22, False), (TOP, TOP, 17, True), (TOP, TOP, 24, True),
         (TOP, TOP, 31, True), (TOP, TOP, 32, True), (1 << 16, 1 << 15, 40, True)]


def _module_inputs(d, rows):
    rng = np.random.default_rng(d + rows)
    z = np.clip(np.rint(rng.normal(0.0, 48.0, size=(rows, d))), -128, 127).astype(np.int8)
    z[0, :8] = [-128, 127, -127, 0, -128, 1, -1, 126]
    return z


@pytest.mark.gpu
@pytest.mark.parametrize("m_z,m_y,n,wide", FORMS)
def test_residual_forms(gpu_lib, m_z, m_y, n, wide):
    assert wide == (n > 31 or (m_z + m_y) * 128 + (1 << (n - 1)) >= 1 << 31)
    new = {"m_z": m_z, "m_y": m_y, "shift_r": n}
    label = f"m_z={m_z} m_y={m_y} n={n}"
    d = 256
    z = _module_inputs(d, 150)
    _check_ffn(gpu_lib, dataclasses.replace(make_ffn(d, "calibrated", seed=5, S_z=1.0 / 32), **new), z, label)
    _check_conv(gpu_lib, dataclasses.replace(make_conv(d, "calibrated", seed=6, S_z=1.0 / 32), **new),
                z.reshape(3, 50, d), [50, 1, 33], label)
    blk = make_workload("tiny", "calibrated").blocks[0]
    blk.x[0, 0, :8] = z[0, :8]
    _check_mhsa(gpu_lib, blk, dataclasses.replace(make_residual(blk, "calibrated", seed=7), **new), label)


@pytest.mark.parametrize("m_z,m_y,n,wide", [f for f in FORMS if f[2] < 31])
def test_forms_are_not_trivial(m_z, m_y, n, wide):
    """The multipliers leave outputs that vary (CPU only): the cases above compare more than zeros."""
    d = 256
    f = dataclasses.replace(make_ffn(d, "calibrated", seed=5, S_z=1.0 / 32), m_z=m_z, m_y=m_y, shift_r=n)
    assert len(np.unique(core.ffn_module(f, _module_inputs(d, 150)))) >= 3
