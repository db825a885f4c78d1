"""Every length with a mixed-radix compile-time plan, along x and along z.

Rows and columns of each length (odd ones, one and more transforms a block,
an odd number of rows, so that the last has no partner), in FP64 and in FP32
spectra with refinement, against the oracle with the suite's tolerances
(parity_util.check).
"""
import numpy as np
import pytest

import parity_util as PU
from paper_2103_01874_amd import binding, synth
from test_gpu_configs import run_single

pytestmark = pytest.mark.gpu

LENGTHS = [18, 24, 27, 36, 48, 54, 72, 81, 108, 144, 162, 216, 243, 288, 324, 432, 486, 768]


@pytest.mark.parametrize("precision", [binding.PPE_PREC_FP64, binding.PPE_PREC_MIXED])
@pytest.mark.parametrize("n", LENGTHS)
def test_mixed_radix_lengths(n, precision):
    for shape, ybc in (((n, 5, 3), 0), ((9, 7, n), 1)):
        pr = synth.random_problem(*shape, seed=9800 + n, ybc=ybc)
        got, rec = (run_single(pr, precision, 0) if precision == binding.PPE_PREC_FP64
                    else run_single(pr, precision, 3, tol=1e-13))
        PU.check(pr, got, rec, PU.oracle_step(pr), label=f"{shape} ybc={ybc} ")


LONG = [576, 648, 729, 864, 972, 1152, 1296, 1458, 1536, 1728, 1944]


@pytest.mark.parametrize("precision", [binding.PPE_PREC_FP64, binding.PPE_PREC_MIXED])
@pytest.mark.parametrize("n", LONG)
def test_long_mixed_radix_lengths(n, precision):
    test_mixed_radix_lengths(n, precision)
