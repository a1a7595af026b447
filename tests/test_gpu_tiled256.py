"""The 256-token tiles at their edges: every tile height (32 to 256 rows, one row tile and several), one row more and
less than a tile, k of one to five steps, tokens one more and less than a tile.  Logits, log-sum-exps and
cross-entropy against a float64 product."""
import numpy as np
import pytest
import torch

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.gpu


def _bound(h, W, d, tau):
    """bf16 products are exact in binary32; d sums in any order and one multiplication by 1/tau."""
    return (d + 2) * 2.0 ** -24 * (h.abs() @ W.abs().t()) * tau + 1e-30


@pytest.mark.parametrize("B,K,d,V", [
    (1, 8, 64, 255), (1, 16, 320, 257), (17, 1, 64, 300), (8, 4, 128, 511), (3, 11, 192, 256), (6, 8, 64, 1000),
    (7, 7, 256, 513), (8, 8, 320, 255), (13, 5, 128, 257), (5, 16, 64, 700), (9, 9, 128, 258), (14, 8, 192, 260), (96, 1, 192, 256), (97, 1, 256, 513), (8, 16, 320, 300), (43, 3, 64, 511),
    (10, 16, 128, 259), (23, 7, 192, 64), (48, 4, 256, 1024), (193, 1, 64, 270), (15, 15, 128, 258), (16, 16, 192, 769),
    (257, 1, 64, 33), (32, 12, 128, 900), (43, 3, 1024, 511), (23, 7, 1088, 264), (193, 1, 1024, 300), (15, 15, 1152, 258),
    (16, 16, 960, 257), (17, 16, 1024, 256), (32, 12, 1088, 513),
])
def test_logits_and_lse(B, K, d, V):
    g = torch.Generator().manual_seed(B * 100 + K)
    W = (torch.randn(V, d, generator=g) * 0.1).bfloat16()
    hd, ht = torch.randn(B, K, d, generator=g).bfloat16(), torch.randn(B, K, d, generator=g).bfloat16()
    vs = fb.VerifyStep(B, K, max(K, 4), d, V, diag=True, diag_logits=True, gemm_variant=fb.FEF_GEMM_TILED256)
    vs(hd.cuda(), ht.cuda(), W.cuda(), 5, temperature=0.7)
    torch.cuda.synchronize()
    h, W64 = torch.cat([hd.reshape(-1, d), ht.reshape(-1, d)]).double(), W.double()
    tau = float(np.float32(1.0) / np.float32(0.7))
    want, bound = (h @ W64.t()) * tau, _bound(h, W64, d, tau)
    got = vs.diag["logits"].double().cpu().reshape(-1, V)
    assert bool(((got - want).abs() <= bound).all())
    lse = vs.diag["lse"].double().cpu().reshape(-1)
    # 1e-5: exp, log and sums of at most 1024 terms at magnitudes below 64
    assert bool(((lse - torch.logsumexp(want, 1)).abs() <= bound.max(1).values + 1e-5).all())


@pytest.mark.parametrize("R,d,V", [(129, 64, 257), (193, 128, 255), (257, 64, 300), (320, 192, 512), (321, 64, 600),
                                   (385, 128, 256), (449, 64, 1000), (513, 320, 31), (769, 64, 258), (300, 1024, 259), (321, 1088, 300), (449, 1024, 513), (513, 1152, 255)])
def test_cross_entropy(R, d, V):
    g = torch.Generator().manual_seed(R)
    W, h = (torch.randn(V, d, generator=g) * 0.1).bfloat16(), torch.randn(R, d, generator=g).bfloat16()
    labels = torch.randint(0, V, (R,), generator=g, dtype=torch.int32)
    labels[::5] = V - 1
    labels[3] = -1
    ce, loss = fb.HeadCrossEntropy(R, d, V)(h.cuda(), W.cuda(), labels.cuda())
    L = h.double() @ W.double().t()
    want = torch.logsumexp(L, 1) - L.gather(1, labels.long().clamp(min=0)[:, None])[:, 0]
    want[3] = 0.0
    bound = 2 * _bound(h.double(), W.double(), d, 1.0).max(1).values + 1e-5
    assert bool(((ce.double().cpu() - want).abs() <= bound).all())
    assert abs(float(loss) - float(want.sum())) <= float(bound.sum())
