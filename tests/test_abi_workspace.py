"""fef_workspace_bytes does not depend on the phase: a caller who sizes a workspace once may run whole rounds, split rounds
and baseline steps with it.  Decided on the host; no GPU needed."""
import os

import pytest

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.skipif(not os.path.exists(fb.LIB_PATH), reason="libfef.so not built")


def _sizes(p, K):
    out = []
    for p.phase in (fb.FEF_PHASE_FUSED, fb.FEF_PHASE_DRAFT, fb.FEF_PHASE_TARGET):
        out.append(fb.fef_workspace_bytes(p, K, 64))
    return out


@pytest.mark.parametrize("d", [512, 1088, 4096])
@pytest.mark.parametrize("V", [300, 5000, 32000, 50257, 66000, 100003, 126464, 151936])
def test_one_size_for_all_phases(d, V):
    for B in (1, 2, 3, 4, 6, 8, 10, 13, 16, 20, 33, 64):
        for K in (1, 4, 8, 16):
            fused, draft, target = _sizes(fb.make_params(B, d, V), K)
            assert fused > 0 and fused == draft == target, (B, K)


def test_a_variant_that_serves_only_the_halves():
    # 2 B K = 160 rows are more than STREAM takes, B K = 80 are not
    fused, draft, target = _sizes(fb.make_params(10, 512, 5000, gemm_variant=fb.FEF_GEMM_STREAM), 8)
    assert fused == 0 and draft == target > 0
