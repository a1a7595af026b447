"""The 256-token tile kernel where a workgroup's tokens are not one whole tile: runs of 16- and 64-token units over several
tiles, equal shares of 32 to 256 tokens in the cross-entropy, and whole tiles beside partly filled ones, at every tile
height (32 to 256 rows) and one row to either side of it.  Logits, log-sum-exps, cross-entropy against a float64 product."""
import numpy as np
import pytest
import torch

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.gpu

# shares of one to eight units of 32 tokens (8200: 1 and 2; 16500: 2 and 3; 33001: 4 and 5; 50257: 6 and 7; 65536: 8), a
# second round (66000, 100003); for the runs one tile per workgroup, one and a part, two and a part
VOCABULARIES = [8200, 16500, 33001, 50257, 65535, 66000, 100003, 135000]


def _bound(h, W, d, tau):
    """bf16 products are exact in binary32; d sums in any order and one multiplication by 1/tau."""
    return (d + 2) * 2.0 ** -24 * (h.abs() @ W.abs().t().contiguous()) * tau + 1e-30


def _check_round(variant, M, d, V):
    g = torch.Generator(device="cuda").manual_seed(M * 7 + V)
    B, K = (M // 2, 1)
    W = (torch.randn(V, d, generator=g, device="cuda") * 0.1).bfloat16()
    hd, ht = (torch.randn(B, K, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    vs = fb.VerifyStep(B, K, 4, d, V, diag=True, diag_logits=True, gemm_variant=variant)
    vs(hd, ht, W, 5, temperature=0.7)
    h, W64 = torch.cat([hd.reshape(-1, d), ht.reshape(-1, d)]).double(), W.double()
    tau = float(np.float32(1.0) / np.float32(0.7))
    want, bound = (h @ W64.t().contiguous()) * tau, _bound(h, W64, d, tau)
    assert bool(((vs.diag["logits"].view(-1, V) - want).abs() <= bound).all())
    # 2e-5: exp, log and sums of at most 135000 terms (two levels of at most 640) at magnitudes below 64
    assert bool(((vs.diag["lse"].view(-1) - torch.logsumexp(want, 1)).abs() <= bound.max(1).values + 2e-5).all())


def _check_loss(R, d, V):
    g = torch.Generator(device="cuda").manual_seed(R + V)
    W = (torch.randn(V, d, generator=g, device="cuda") * 0.1).bfloat16()
    h = torch.randn(R, d, generator=g, device="cuda").bfloat16()
    labels = torch.randint(0, V, (R,), generator=g, device="cuda", dtype=torch.int32)
    ce, _ = fb.HeadCrossEntropy(R, d, V)(h, W, labels)
    L = h.double() @ W.double().t().contiguous()
    want = torch.logsumexp(L, 1) - L.gather(1, labels.long()[:, None])[:, 0]
    bound = 2 * _bound(h.double(), W.double(), d, 1.0).max(1).values + 2e-5
    assert bool(((ce - want).abs() <= bound).all())


@pytest.mark.parametrize("V", VOCABULARIES)
@pytest.mark.parametrize("variant,d", [(fb.FEF_GEMM_STREAM, 64), (fb.FEF_GEMM_STREAM, 192), (fb.FEF_GEMM_ROWSTREAM, 512)])
def test_runs(variant, d, V):
    for M in (2, 32, 34, 64, 66, 96, 98, 126, 128):
        _check_round(variant, M, d, V)


@pytest.mark.parametrize("V", [8200, 33001, 65535, 100003])
def test_whole_tiles_of_one_row_tile(V):
    for M in (32, 34, 96, 128, 130, 160, 162, 190, 194, 224, 226, 254, 256):
        _check_round(fb.FEF_GEMM_TILED256, M, 128, V)


@pytest.mark.parametrize("V", VOCABULARIES)
def test_shares_of_a_cross_entropy_call(V):
    for R in (1, 31, 33, 64, 65, 95, 97, 128, 129, 160, 161, 191, 193, 224, 225, 255, 256):
        d = 64 + 64 * (R % 3)
        g = torch.Generator(device="cuda").manual_seed(R + V)
        W = (torch.randn(V, d, generator=g, device="cuda") * 0.1).bfloat16()
        h = torch.randn(R, d, generator=g, device="cuda").bfloat16()
        labels = torch.randint(0, V, (R,), generator=g, device="cuda", dtype=torch.int32)
        labels[::5] = V - 1
        ce, loss = fb.HeadCrossEntropy(R, d, V)(h, W, labels)
        L = h.double() @ W.double().t().contiguous()
        want = torch.logsumexp(L, 1) - L.gather(1, labels.long()[:, None])[:, 0]
        bound = 2 * _bound(h.double(), W.double(), d, 1.0).max(1).values + 2e-5
        assert bool(((ce - want).abs() <= bound).all()), R
        assert abs(float(loss) - float(want.sum())) <= float(bound.sum())


@pytest.mark.parametrize("V", [257, 2000, 8437, 16384, 32700])  # 2 to 128 token tiles: more row tiles than the rows take
@pytest.mark.parametrize("variant,d,rows", [(fb.FEF_GEMM_STREAM, 192, (66, 96, 126, 128)), (fb.FEF_GEMM_ROWSTREAM, 512, (66, 100, 128)),
                                            (fb.FEF_GEMM_TILED256, 128, (66, 130, 190, 200, 256, 258, 300, 450, 528, 770, 1000))])
def test_more_row_tiles_where_the_vocabulary_is_short(variant, d, rows, V):
    for M in rows:
        _check_round(variant, M, d, V)


@pytest.mark.parametrize("V", [257, 8437, 16384, 40000])
@pytest.mark.parametrize("R", [200, 257, 300, 512, 513, 1000])
@pytest.mark.parametrize("d", [128, 1024, 1088])  # eight and four wavefronts
def test_row_tiles_of_a_cross_entropy_call(V, R, d):
    _check_loss(R, d, V)


@pytest.mark.parametrize("R,d", [(300, 4096), (300, 4160), (384, 4096), (385, 3072), (385, 3136), (512, 3072), (512, 3584)])  # eight or four
def test_two_row_tiles_of_a_cross_entropy_call(R, d):
    _check_loss(R, d, 50257)


# 288 MiB of W and a row, or 64 columns, more: ordinary and non-temporal loads.  One row tile at every height that a form has (one or two in a
# cross-entropy call of more than 256 rows); that these calls take the forms they are meant for is checked in test_head_rules.py.
LINE_OF_A_ROUND = [(73728, 2048), (73729, 2048)]
ROUNDS_AT_THE_LINE = [(fb.FEF_GEMM_STREAM, (2, 34, 66, 128)), (fb.FEF_GEMM_ROWSTREAM, (2, 34, 66, 128)),
                      (fb.FEF_GEMM_TILED256, (32, 64, 96, 128, 160, 192, 224, 256))]
LINES_OF_A_LOSS = [(126464, (1152, 1216), (30, 60, 90, 120, 150, 190, 220, 250, 300, 380, 440, 512)),  # whole tiles
                   (65537, (2240, 2304), (30, 120, 250))]                                              # shares


@pytest.mark.parametrize("variant,rows", ROUNDS_AT_THE_LINE)
@pytest.mark.parametrize("V,d", LINE_OF_A_ROUND)
def test_w_to_either_side_of_the_line_for_non_temporal_loads(variant, rows, V, d):
    for M in rows:
        _check_round(variant, M, d, V)


# (runs of 257 to 320 tokens, as those are, take head_runs_kernel; these stay in the tile kernel)
TILES_AT_THE_LINE = [(fb.FEF_GEMM_STREAM, (2, 34, 66, 128)), (fb.FEF_GEMM_ROWSTREAM, (2, 34, 66, 128))]


@pytest.mark.parametrize("variant,rows", TILES_AT_THE_LINE)
@pytest.mark.parametrize("V", [36864, 36865])
def test_runs_of_one_tile_to_either_side_of_that_line(variant, rows, V):
    for M in rows:
        _check_round(variant, M, 4096, V)


@pytest.mark.parametrize("V,d,rows", [(V, d, rows) for V, ds, rows in LINES_OF_A_LOSS for d in ds])
def test_cross_entropy_to_either_side_of_that_line(V, d, rows):
    for R in rows:
        _check_loss(R, d, V)


@pytest.mark.parametrize("variant,M", [(fb.FEF_GEMM_TILED256, 40), (fb.FEF_GEMM_STREAM, 40), (fb.FEF_GEMM_ROWSTREAM, 40),
                                       (fb.FEF_GEMM_TILED256, 200), (fb.FEF_GEMM_TILED256, 300)])
@pytest.mark.parametrize("first,last", [(640, 704), (512, 768), (16, 32), (1000, 3000)])
def test_tokens_of_logit_minus_infinity(variant, M, first, last):
    """Tokens banned by an overflowing column of W: a piece of a tile, or all of it, that holds nothing else brings no mass
    and no NaN, and its neighbours keep theirs."""
    _check_banned(variant, M, 512, 9001, first, last)


# The same where a call takes another kernel or form than those of 9001 tokens do (test_head_rules.py: which): variant, M, d, V
BANNED = {"tiles, runs of 64": (fb.FEF_GEMM_STREAM, 40, 512, 33001), "tiles, runs of 16": (fb.FEF_GEMM_ROWSTREAM, 40, 512, 33001),
          "short runs": (fb.FEF_GEMM_ROWSTREAM, 72, 1024, 20011),
          "double runs of 64": (fb.FEF_GEMM_STREAM, 40, 512, 66000), "double runs of 16": (fb.FEF_GEMM_ROWSTREAM, 40, 512, 70001),
          "pieces of 128": (fb.FEF_GEMM_TILED256, 256, 4096, 16384),
          "H in registers": (fb.FEF_GEMM_SKINNY, 16, 512, 9001), "H in registers, 32 rows": (fb.FEF_GEMM_SKINNY, 32, 512, 9001),
          "H in LDS": (fb.FEF_GEMM_SKINNY, 16, 512, 33001), "H in LDS, 32 rows": (fb.FEF_GEMM_SKINNY, 32, 512, 33001),
          "H in LDS, from any slice": (fb.FEF_GEMM_SKINNY, 16, 2048, 33001), "H in LDS, two tiles": (fb.FEF_GEMM_SKINNY, 32, 512, 100003)}


@pytest.mark.parametrize("first,last", [(640, 704), (512, 768), (16, 32), (1000, 3000)])
@pytest.mark.parametrize("call", list(BANNED))
def test_tokens_of_logit_minus_infinity_in_the_other_kernels(call, first, last):
    _check_banned(*BANNED[call], first, last)


def _check_banned(variant, M, d, V, first, last):
    g = torch.Generator(device="cuda").manual_seed(first)
    W = torch.randn(V, d, generator=g, device="cuda") * 0.1
    W[first:last, 0] = -3e38
    h = torch.randn(M, d, generator=g, device="cuda")
    h[:, 0] = 8.0
    W, h = W.bfloat16(), h.bfloat16()
    vs = fb.VerifyStep(M // 2, 1, 4, d, V, diag=True, diag_logits=True, gemm_variant=variant)
    vs(h[:M // 2].view(M // 2, 1, d), h[M // 2:].view(M // 2, 1, d), W, 1)
    L = h.double() @ W.double().t().contiguous()
    keep = torch.ones(V, dtype=torch.bool, device="cuda")
    keep[first:last] = False
    want, bound = torch.logsumexp(L[:, keep], 1), _bound(h.double(), W.double()[keep], d, 1.0).max(1).values + 2e-5
    assert bool((vs.diag["lse"].view(-1) - want).abs().le(bound).all())
    assert bool((vs.diag["logits"].view(M, V)[:, first:last] == -float("inf")).all())
    drafts = vs.diag["draft_tokens"]
    assert bool(((drafts < first) | (drafts >= last)).all())
