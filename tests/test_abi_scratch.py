"""Which calls fit the built-in scratch of fef_verify_step_static: decided on the host, by a fixed count of partials per
row (at most 256 for the variants up to 128 rows, one per 256 tokens above), whatever tiles the kernel takes."""
import ctypes
import os

import pytest

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.skipif(not os.path.exists(fb.LIB_PATH), reason="libfef.so not built")


def _total(B, K, V, variant):
    BK, M = B * K, 2 * B * K
    partials = {fb.FEF_GEMM_SKINNY: min(256, -(-V // 16)), fb.FEF_GEMM_STREAM: min(256, -(-V // 256)),
                fb.FEF_GEMM_ROWSTREAM: min(256, -(-V // 128)), fb.FEF_GEMM_TILED256: -(-V // 256)}[variant]
    parts = [M * (-(-V // 64) * 64) * 4, M * partials * 8, M * 4, BK * 4, BK * 4, BK * 4, B * 4, B * 536, B * -(-V // 256) * 4]
    return sum(-(-p // 256) * 256 for p in parts)


@pytest.mark.parametrize("B,K,d", [(1, 8, 4096), (3, 8, 4096), (4, 8, 4096), (5, 8, 4096), (7, 8, 1088), (13, 8, 512), (33, 8, 4096)])
def test_limit_of_the_built_in_scratch(B, K, d):
    lib = fb.lib()
    limit, M = fb.FEF_STATIC_SCRATCH_BYTES, 2 * B * K
    top = limit // (4 * M)
    fits = []
    for V in [*range(top - 1500, top + 200, 50), top // 2]:
        p = fb.make_params(B, d, V)
        variant = fb.fef_select_gemm(p, K)
        null = ctypes.c_void_p(0)   # refused for the pointers, if not for the size: nothing is launched
        s = lib.fef_verify_step_static(ctypes.byref(p), null, null, null, K, 32, ctypes.c_uint64(0), null, null, null)
        assert s != fb.FEF_OK
        fits.append(s != fb.FEF_ERR_WORKSPACE)
        assert fits[-1] == (_total(B, K, V, variant) <= limit), (V, variant)
    assert any(fits) and not all(fits)


@pytest.mark.parametrize("phase", [fb.FEF_PHASE_FUSED, fb.FEF_PHASE_DRAFT, fb.FEF_PHASE_TARGET])
@pytest.mark.parametrize("B,K,d", [(1, 8, 4096), (3, 8, 4096), (5, 16, 4096), (5, 8, 4096), (7, 8, 1088), (13, 8, 512), (33, 8, 4096)])
def test_a_workspace_of_that_size_always_fits(B, K, d, phase):
    """What the header promises: fef_workspace_bytes <= FEF_STATIC_SCRATCH_BYTES is never refused for its size."""
    lib, limit = fb.lib(), fb.FEF_STATIC_SCRATCH_BYTES
    top = limit // (8 * B * K)
    below = 0
    for V in [*range(top - 900, top + 100, 4), 51872]:
        p = fb.make_params(B, d, V)
        p.phase = phase
        if fb.fef_workspace_bytes(p, K, 32) > limit:
            continue
        below += 1
        null = ctypes.c_void_p(0)
        s = lib.fef_verify_step_static(ctypes.byref(p), null, null, null, K, 32, ctypes.c_uint64(0), null, null, null)
        assert s not in (fb.FEF_OK, fb.FEF_ERR_WORKSPACE), (V, fb.fef_last_error())   # the pointers; without a GPU the buffer's address
    assert below
