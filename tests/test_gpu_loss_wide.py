"""Cross-entropy of 257 to 320 rows in one row tile (csrc/head_loss.hip) against a float64 product: edges of its rows and shares."""
import pytest

import test_gpu_shares as shares

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [45057, 49152, 50257, 57344])
@pytest.mark.parametrize("d", [64, 128, 192, 1024])
def test_against_a_float64_product(d, V):
    for R in (257, 272, 303, 304) + ((305, 320) if V <= 49152 else ()):
        shares._check_loss(R, d, V)
