"""The fp32 head kernel at the edges of its tiles (64 tokens, 32 or 64 rows, 64 columns of k, float4 or
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
