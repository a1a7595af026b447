"""Runs of STREAM and ROWSTREAM in one walk over k (csrc/head_runs.hip) against the tiles they took before: whole rounds against checksums
recorded then (tests/golden/runs_bits.txt), and logits against a float64 product around the lines of its rules."""
import os

import pytest

from paper_2605_14305_amd import binding as fb
import test_gpu_order as order
import test_gpu_shares as shares

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "runs_bits.txt")
AUTO, STREAM, ROWSTREAM, TILED256 = fb.FEF_GEMM_AUTO, fb.FEF_GEMM_STREAM, fb.FEF_GEMM_ROWSTREAM, fb.FEF_GEMM_TILED256
# kind, variant, B, K, d, V: every tile height, short runs of 16 to 128 tokens, double ones of 257 to 512, starts in the middle of a k-step
CASES = [
    ("fused", AUTO, 3, 8, 1024, 32768), ("greedy", AUTO, 3, 7, 1536, 31001), ("fused", ROWSTREAM, 4, 8, 1536, 16001), ("fused", AUTO, 6, 8, 2048, 8191),
    ("fused", ROWSTREAM, 8, 8, 512, 12289), ("fused", ROWSTREAM, 1, 9, 1536, 129), ("topn", AUTO, 3, 29, 1024, 20011), ("split", AUTO, 9, 4, 1536, 28003),
    ("fused", AUTO, 3, 8, 2048, 81920), ("fused", AUTO, 5, 8, 1024, 70001), ("fused", AUTO, 6, 8, 512, 126464), ("fused", ROWSTREAM, 1, 16, 1024, 66001),
    ("fused", AUTO, 4, 8, 1024, 65537), ("fused", AUTO, 8, 8, 2560, 106496), ("fused", AUTO, 5, 10, 576, 90001), ("fused", AUTO, 1, 17, 1088, 73000),
    ("split", AUTO, 10, 12, 704, 131072), ("topn", AUTO, 4, 16, 64, 100003), ("greedy", AUTO, 4, 12, 512, 69999), ("fused", STREAM, 1, 7, 128, 67001),
    # to either side of the line of short_runs_lag
    ("fused", AUTO, 3, 8, 1024, 20352), ("fused", AUTO, 5, 4, 1024, 20353), ("fused", ROWSTREAM, 1, 8, 1024, 30000), ("fused", ROWSTREAM, 4, 8, 1024, 22000),
    ("fused", AUTO, 11, 3, 1024, 22000),
    # pieces of runs and tiles, partials from the logits (but two calls past the lines of pieces_pay: 176 rows, and V = 32700)
    ("fused", AUTO, 4, 8, 2048, 16001), ("fused", AUTO, 8, 8, 2560, 12289), ("fused", AUTO, 16, 8, 4096, 8437), ("fused", AUTO, 11, 8, 2048, 16384),
    ("fused", TILED256, 2, 8, 2048, 5003), ("fused", STREAM, 1, 9, 2112, 4001), ("fused", AUTO, 4, 8, 3072, 32700), ("split", AUTO, 12, 8, 2048, 9001),
    ("topn", AUTO, 5, 20, 2048, 15001), ("greedy", AUTO, 9, 8, 2048, 777), ("fused", AUTO, 3, 7, 2048, 15), ("fused", AUTO, 6, 8, 3584, 14001),
    # to either side of the lines of whole tiles in pieces
    ("fused", AUTO, 14, 8, 2048, 9000), ("fused", AUTO, 15, 8, 2048, 9000), ("fused", AUTO, 16, 8, 512, 4097), ("fused", AUTO, 16, 8, 512, 4096),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_rounds_to_the_last_bit(case):
    with open(GOLDEN) as f:
        golden = {tuple(r[:6]): r[6:] for r in (line.split() for line in f if not line.startswith("#"))}
    assert dict(zip(order.COLUMNS, order.checksums(fb, *case))) == dict(zip(order.COLUMNS, golden[tuple(map(str, case))]))


@pytest.mark.parametrize("variant,d,V", [(ROWSTREAM, 512, 24576), (ROWSTREAM, 512, 24577), (ROWSTREAM, 1024, 32768), (ROWSTREAM, 1024, 17), (ROWSTREAM, 512, 65537),
                                         (STREAM, 64, 65537), (STREAM, 192, 98305), (STREAM, 1088, 81920), (ROWSTREAM, 512, 131072)])
def test_against_a_float64_product(variant, d, V):
    for M in (2, 16, 32, 34, 64, 66, 96, 98, 128):
        shares._check_round(variant, M, d, V)


# Every shape of a piece (test_head_rules.py: which): tokens and rows of 64 and 128, both row tiles partly filled.  variant, d, V, rows
PIECES = [(STREAM, 2112, 12289, (34, 64, 66, 128)), (ROWSTREAM, 2048, 12289, (34, 64, 66, 128)), (STREAM, 2112, 16384, (66, 98, 128)), (ROWSTREAM, 2048, 16383, (66, 98, 128)),
          (TILED256, 2560, 12288, (130, 192)), (TILED256, 4096, 16384, (194, 256)), (TILED256, 2048, 10240, (130, 192)), (TILED256, 2048, 8437, (66, 128, 130, 256)),
          (TILED256, 2112, 4001, (130, 192, 256)), (STREAM, 576, 5119, (10, 64)), (ROWSTREAM, 512, 5120, (10, 128))]


@pytest.mark.parametrize("variant,d,V,rows", PIECES)
def test_every_shape_of_a_piece_against_a_float64_product(variant, d, V, rows):
    for M in rows:
        shares._check_round(variant, M, d, V)


@pytest.mark.parametrize("variant,d,V", [(STREAM, 2112, 16384), (STREAM, 2112, 32768), (STREAM, 2048, 129), (ROWSTREAM, 2048, 16383), (ROWSTREAM, 2048, 31), (TILED256, 2048, 16384),
                                         (TILED256, 2112, 257)])
def test_pieces_against_a_float64_product(variant, d, V):
    for M in (2, 34, 64, 66, 128) + ((130, 192, 194, 256) if variant == TILED256 else ()):
        shares._check_round(variant, M, d, V)
