"""Row counts at which a launch would reach 2^32 threads: the calls below are within the documented limits and have to run."""
import pytest
import torch

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.gpu


def test_diagnostic_logits_of_2_to_24_rows():
    B, K, d, V = 1 << 17, 64, 64, 3
    W = torch.randn(V, d, device="cuda").bfloat16()
    hd, ht = (torch.randn(B, K, d, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    vs = fb.VerifyStep(B, K, K, d, V, diag=True, diag_logits=True)
    vs.diag["logits"].fill_(float("nan"))
    vs(hd, ht, W, 1)
    torch.cuda.synchronize()
    for got, h in zip(vs.diag["logits"].view(2, -1, V), (hd, ht)):
        for x, y in zip(got.split(1 << 20), h.view(-1, d).split(1 << 20)):
            want = y.double() @ W.double().t().contiguous()
            # 64 products and sums in binary32, magnitudes of the products below 64 together
            assert bool(((x - want).abs() <= 66 * 2.0 ** -24 * 512).all())
    del vs
    torch.cuda.empty_cache()


def test_cross_entropy_of_2_to_22_rows_with_a_small_hidden_size():
    R, d, V = (1 << 22) + 5, 64, 131072
    W = torch.randn(V, d, device="cuda").mul_(0.3).bfloat16()
    h = torch.randn(R, d, device="cuda", dtype=torch.bfloat16)
    labels = torch.randint(0, V, (R,), device="cuda", dtype=torch.int32)
    ce, _ = fb.HeadCrossEntropy(R, d, V)(h, W, labels)
    torch.cuda.synchronize()
    rows = torch.tensor([0, 1, 255, 256, 12345, R // 2, R - 257, R - 2, R - 1], device="cuda")
    L = h[rows].double() @ W.double().t().contiguous()
    want = torch.logsumexp(L, 1) - L.gather(1, labels[rows].long()[:, None])[:, 0]
    # two terms of 66 half-ulps of products of magnitude below 64 together, and 1e-5 for exp, log and their sums
    assert bool(((ce[rows].double() - want).abs() <= 2 * 66 * 2.0 ** -24 * 64 + 1e-5).all())
    assert bool(torch.isfinite(ce).all())
    torch.cuda.empty_cache()
