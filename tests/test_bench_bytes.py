"""bench.py prices a head launch by the bytes it cannot do without; its count of partials per row has to be the library's,
which shows in the workspace that the library asks for."""
import ctypes
import os

import pytest

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.skipif(not os.path.exists(fb.LIB_PATH), reason="libfef.so not built")
bench = pytest.importorskip("bench")


@pytest.mark.parametrize("R", [32, 64, 128, 256, 288, 2048])
@pytest.mark.parametrize("V", [31, 200, 2000, 8192, 32000, 50257, 51201, 66000, 100003, 126464, 151936])
def test_partials_of_a_cross_entropy_call(V, R):
    got = fb.lib().fef_cross_entropy_workspace_bytes(ctypes.byref(fb.make_params(1, 512, V)), R)
    assert got == R * bench.ce_tiles(V, R) * 8 + -(-R * 4 // 256) * 256   # R * 8 is a multiple of 256


@pytest.mark.parametrize("B,K,d,name", [(1, 8, 4096, "skinny"), (1, 8, 1088, "stream"), (4, 8, 4096, "stream"), (3, 8, 512, "rowstream"),
                                        (16, 8, 4096, "tiled256"), (64, 8, 4096, "tiled256")])
@pytest.mark.parametrize("V", [200, 2000, 32000, 50257, 100003, 126464, 151936])
def test_partials_of_a_verify_step(V, B, K, d, name):
    p = fb.make_params(B, d, V)
    assert {"skinny": fb.FEF_GEMM_SKINNY, "stream": fb.FEF_GEMM_STREAM, "rowstream": fb.FEF_GEMM_ROWSTREAM,
            "tiled256": fb.FEF_GEMM_TILED256}[name] == fb.fef_select_gemm(p, K)
    BK, M = B * K, 2 * B * K
    # the halves of a split round share the workspace and may leave more partials per row
    p.phase = fb.FEF_PHASE_DRAFT
    of = {fb.FEF_GEMM_SKINNY: "skinny", fb.FEF_GEMM_STREAM: "stream", fb.FEF_GEMM_ROWSTREAM: "rowstream", fb.FEF_GEMM_TILED256: "tiled256"}
    most = max(bench.head_partials(V, name), bench.head_partials(V, of[fb.fef_select_gemm(p, K)]))
    parts = [M * (-(-V // 64) * 64) * 4, M * most * 8, M * 4, BK * 4, BK * 4, BK * 4, B * 4, B * 536, B * -(-V // 256) * 4]
    assert fb.fef_workspace_bytes(p, K, 64) == sum(-(-x // 256) * 256 for x in parts)
