"""The nibble operand around its layout blocks of 512 samples (32 words of 16):
every pair's sums against the oracle, with and without a sample list."""
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_ld_nibbles import FORCE, MFMA, _check, _codes

import numpy as np


@pytest.mark.parametrize("path", [MFMA, FORCE])
@pytest.mark.parametrize("n", [511, 512, 513, 1023, 1025])
def test_around_512_samples(n, path):
    assert _check(_codes(67, n, n), 66, path) > 0


@pytest.mark.parametrize("m", [511, 512, 513])
def test_around_512_listed_samples(m):
    idx = np.random.default_rng(m).permutation(900)[:m]
    assert _check(_codes(65, 900, m), 64, MFMA, idx=idx) > 0
