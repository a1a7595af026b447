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
