"""The kernel that serves up to 32 rows of a long vocabulary (csrc/head_slices.hip) against the one with H in registers, whose order of
sums it keeps: logits to the bit against the same columns in a vocabulary that the other kernel serves, and whole rounds against
checksums recorded when that kernel served them all (tests/golden/slices_bits.txt)."""
import os

import pytest
import torch

from paper_2605_14305_amd import binding as fb
import test_gpu_order as order
import test_gpu_shares as shares

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "slices_bits.txt")
SKINNY, AUTO = fb.FEF_GEMM_SKINNY, fb.FEF_GEMM_AUTO
# kind, variant, B, K, d, V: every hidden size, one and two groups of 16 rows, one to five tiles per run, a partly filled last one, W
# by ordinary and by non-temporal loads
CASES = [
    ("fused", SKINNY, 1, 8, 512, 32769), ("fused", SKINNY, 1, 16, 512, 65537), ("greedy", SKINNY, 2, 8, 512, 300001), ("fused", SKINNY, 1, 1, 1024, 40000),
    ("topn", AUTO, 1, 32, 1024, 65536), ("fused", SKINNY, 1, 16, 1024, 150001), ("fused", SKINNY, 1, 8, 2048, 100003), ("fused", SKINNY, 1, 13, 2048, 33000),
    ("split", AUTO, 1, 20, 2560, 50257), ("fused", SKINNY, 1, 7, 2560, 131073), ("fused", SKINNY, 1, 9, 3072, 48001), ("fused", SKINNY, 1, 8, 3584, 151936),
    ("topn", AUTO, 1, 17, 3584, 36007), ("fused", SKINNY, 2, 8, 4096, 32784), ("fused", SKINNY, 1, 8, 4096, 126464), ("split", AUTO, 2, 8, 4096, 37777),
    # to either side of the lines of slices_lag
    ("fused", SKINNY, 1, 16, 512, 81920), ("fused", SKINNY, 1, 7, 512, 81921), ("topn", AUTO, 1, 32, 1024, 65152), ("fused", SKINNY, 1, 16, 2048, 65536),
    ("fused", SKINNY, 1, 8, 2048, 65537), ("fused", SKINNY, 1, 16, 2048, 73729),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_rounds_to_the_last_bit(case):
    with open(GOLDEN) as f:
        golden = {tuple(r[:6]): r[6:] for r in (line.split() for line in f if not line.startswith("#"))}
    assert dict(zip(order.COLUMNS, order.checksums(fb, *case))) == dict(zip(order.COLUMNS, golden[tuple(map(str, case))]))


@pytest.mark.parametrize("d", [512, 1024, 2048, 2560, 3072, 3584, 4096])
def test_logits_as_in_a_short_vocabulary(d):
    V, part = 33001 + d, 32768
    for M in (2, 16, 18, 32):
        g = torch.Generator(device="cuda").manual_seed(M + d)
        W = (torch.randn(V, d, generator=g, device="cuda") * 0.1).bfloat16()
        h = [torch.randn(M // 2, 1, d, generator=g, device="cuda").bfloat16() for _ in range(2)]

        def logits(W):
            vs = fb.VerifyStep(M // 2, 1, 4, d, W.shape[0], diag=True, diag_logits=True, gemm_variant=SKINNY)
            vs(*h, W, 5, temperature=0.7)
            return vs.diag["logits"].view(M, -1)
        whole = logits(W)
        assert torch.equal(whole[:, :part], logits(W[:part])) and torch.equal(whole[:, V - part:], logits(W[V - part:].contiguous()))


@pytest.mark.parametrize("V", [32769, 50257, 65535, 66000, 135000])
@pytest.mark.parametrize("d", [512, 2048])
def test_against_a_float64_product(d, V):
    for M in (2, 14, 16, 18, 30, 32):
        shares._check_round(SKINNY, M, d, V)
