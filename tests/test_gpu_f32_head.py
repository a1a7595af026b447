"""The fp32 head kernel at the edges of its tiles (64 tokens, 16 to 64 rows, 32 columns of k, float4 or
scalar rows): logits and log-sum-exps against a float64 product."""
import numpy as np
import pytest
import torch

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K,d,V", [
    (1, 1, 1, 1), (1, 2, 3, 15), (1, 4, 64, 32), (2, 4, 63, 64), (1, 8, 65, 65), (2, 8, 128, 127),
    (1, 16, 1024, 1000), (3, 6, 599, 517), (4, 8, 100, 130), (5, 9, 68, 200), (33, 1, 66, 77), (13, 5, 256, 64),
])
def test_f32_logits_and_lse(B, K, d, V):
    g = torch.Generator().manual_seed(B * 1000 + d)
    W = torch.randn(V, d, generator=g)
    hd, ht = torch.randn(B, K, d, generator=g), torch.randn(B, K, d, generator=g)
    vs = fb.VerifyStep(B, K, max(K, 4), d, V, dtype="f32", diag=True, diag_logits=True)
    vs(hd.cuda(), ht.cuda(), W.cuda(), 5, temperature=0.7)
    torch.cuda.synchronize()
    h = torch.cat([hd.reshape(-1, d), ht.reshape(-1, d)]).double()
    tau = float(np.float32(1.0) / np.float32(0.7))
    want = (h @ W.double().t()) * tau
    # d products and sums in binary32 in any order, one multiplication by 1/tau: (d + 2) half-ulps of the sum of magnitudes
    bound = (d + 2) * 2.0 ** -24 * (h.abs() @ W.double().abs().t()) * tau + 1e-30
    got = vs.diag["logits"].double().cpu().reshape(-1, V)
    assert bool(((got - want).abs() <= bound).all())
    # log-sum-exp: the logits' bound, and 1e-5 for exp, log and sums of at most 1000 terms at magnitudes below 64
    lse = vs.diag["lse"].double().cpu().reshape(-1)
    assert bool(((lse - torch.logsumexp(want, 1)).abs() <= bound.max(1).values + 1e-5).all())


@pytest.mark.parametrize("R,d,V", [(1, 5, 3), (33, 64, 129), (70, 130, 64)])
def test_f32_cross_entropy(R, d, V):
    g = torch.Generator().manual_seed(R)
    W, h = torch.randn(V, d, generator=g), torch.randn(R, d, generator=g)
    labels = torch.randint(0, V, (R,), generator=g, dtype=torch.int32)
    labels[R // 2] = V - 1
    ce, loss = fb.HeadCrossEntropy(R, d, V, dtype="f32")(h.cuda(), W.cuda(), labels.cuda())
    L = h.double() @ W.double().t()
    want = torch.logsumexp(L, 1) - L.gather(1, labels.long()[:, None])[:, 0]
    bound = 2 * (d + 2) * 2.0 ** -24 * (h.double().abs() @ W.double().abs().t()).max(1).values + 1e-5
    assert bool(((ce.double().cpu() - want).abs() <= bound).all())
    assert abs(float(loss) - float(want.sum())) <= float(bound.sum())


def _check_rows(M, d, V):
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + d)
    W, h = torch.randn(V, d, generator=g, device="cuda"), torch.randn(M, d, generator=g, device="cuda")
    vs = fb.VerifyStep(M // 2, 1, 4, d, V, dtype="f32", diag=True, diag_logits=True)
    vs(h[:M // 2].view(M // 2, 1, d), h[M // 2:].clone().view(M // 2, 1, d), W, 5)
    want = h.double() @ W.double().t().contiguous()
    bound = (d + 2) * 2.0 ** -24 * (h.double().abs() @ W.double().abs().t().contiguous()) + 1e-30  # as above
    assert bool(((vs.diag["logits"].view(M, V) - want).abs() <= bound).all())
    assert bool(((vs.diag["lse"].view(M) - torch.logsumexp(want, 1)).abs() <= bound.max(1).values + 1e-5).all())


@pytest.mark.parametrize("d", [1, 4, 28, 31, 32, 33, 60, 64, 68, 95, 97, 128, 131])  # one to five steps of 32 columns
def test_f32_edges_of_steps(d):
    for M in (2, 16, 18, 34, 50):
        _check_rows(M, d, 257)


@pytest.mark.parametrize("V", [15297, 15360, 15361])  # 240 token tiles and one more
def test_f32_row_tiles(V):
    for M in (14, 16, 18, 32, 34, 48, 50, 64, 66, 96, 130):
        _check_rows(M, 37, V)


@pytest.mark.parametrize("d", [1, 2, 31, 33, 63, 65, 95, 97, 127, 129, 1027])  # 4-byte pieces, 48 and 64 rows: two stages, one to 33 steps
def test_f32_steps_of_many_rows_in_single_pieces(d):
    for M in (34, 48, 50, 64, 98, 130):
        _check_rows(M, d, 32705)


@pytest.mark.parametrize("d", [764, 768, 772, 1024, 1028, 1052, 1056, 1060, 1084, 1092, 1116, 1148, 2004])  # steps of 64 columns where lines are shared
def test_f32_steps_of_64_columns(d):
    for M in (16, 18, 32, 34):
        _check_rows(M, d, 32705)


@pytest.mark.parametrize("d,V", [(1024, 73728), (1024, 73729), (1056, 71494), (1023, 73900), (1028, 73500)])  # 288 MiB of W and more
def test_f32_to_either_side_of_the_line_for_non_temporal_loads(d, V):
    for M in (16, 32, 48, 64):
        _check_rows(M, d, V)


@pytest.mark.parametrize("V", [5, 65])  # the 64th row of a tile starts just under 4 GiB behind the first, and past it from 2^24 + 1 on
@pytest.mark.parametrize("d", [(1 << 24) - 1, 1 << 24, (1 << 24) + 1])
def test_f32_rows_of_two_to_the_24(d, V):
    at = torch.tensor([0, 5, d // 2, d - 2, d - 1], device="cuda")  # few terms, so that the bound means something
    W = torch.zeros(V, d, device="cuda").normal_()
    h = torch.zeros(4, d, device="cuda")
    h[:, at] = torch.randn(4, 5, device="cuda")
    vs = fb.VerifyStep(2, 1, 4, d, V, dtype="f32", diag=True, diag_logits=True)
    vs(h[:2].view(2, 1, d), h[2:].clone().view(2, 1, d), W, 5)
    terms = h[:, None, at].double() * W[None][:, :, at].double()
    assert bool(((vs.diag["logits"].view(4, V) - terms.sum(2)).abs() <= 7 * 2.0 ** -24 * terms.abs().sum(2)).all())
    del W, h, vs
    torch.cuda.empty_cache()
