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


def test_masses_and_logits_of_2_to_24_slots():
    B, K, d, V = 1 << 18, 64, 64, 3
    W = torch.randn(V, d, device="cuda").mul_(0.2).bfloat16()
    hd, ht = (torch.randn(B, K, d, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    vs = fb.VerifyStep(B, K, K, d, V, diag=True, diag_logits=True)
    for t in vs.diag.values():
        t.fill_(-1)
    vs(hd, ht, W, 1)
    torch.cuda.synchronize()
    logits, alpha, resid = vs.diag["logits"].view(2, -1, V), vs.diag["alpha"].view(-1), vs.diag["resid_mass"].view(-1)
    for i in range(0, B * K, 1 << 20):
        law = []
        for half, h in enumerate((hd, ht)):
            want = h.view(-1, d)[i:i + (1 << 20)].double() @ W.double().t().contiguous()
            assert bool(((logits[half, i:i + (1 << 20)] - want).abs() <= 66 * 2.0 ** -24 * 64).all())  # magnitudes below 64 together
            law.append(torch.softmax(want, 1))
        # probabilities: the logits' bound, and 1e-5 for exp, log and their sums
        assert bool(((alpha[i:i + (1 << 20)] - torch.minimum(*law).sum(1)).abs() <= 4 * 66 * 2.0 ** -24 * 64 + 1e-5).all())
        assert bool(((resid[i:i + (1 << 20)] - (law[1] - law[0]).clamp(min=0).sum(1)).abs() <= 4 * 66 * 2.0 ** -24 * 64 + 1e-5).all())
    del vs
    torch.cuda.empty_cache()


def test_masses_of_a_vocabulary_of_more_than_65535_groups_of_chunks():
    V = 65535 * 8 * 256 + 3000  # 8 chunks of 256 tokens per workgroup
    W = torch.randn(V, 1, device="cuda")
    W[-2000:] += 30  # nearly all of the mass at the end
    hd, ht = (torch.full((1, 1, 1), x, device="cuda") for x in (1.0, 0.9))
    vs = fb.VerifyStep(1, 1, 1, 1, V, dtype="f32", diag=True)
    vs.diag["alpha"].fill_(-1)
    vs.diag["resid_mass"].fill_(-1)
    tokens, accepted, _ = vs(hd, ht, W, 3)
    q, p = (torch.softmax(W.view(-1).double() * float(h), 0) for h in (hd, ht))
    # logits below 64 and log-sum-exps round by 2^-19 each, so every law by 2^-17 of itself; 1e-5 for exp, log and the sums of one sign
    assert abs(float(vs.diag["alpha"]) - float(torch.minimum(p, q).sum())) < 2 * 2.0 ** -17 + 1e-5
    assert abs(float(vs.diag["resid_mass"]) - float((p - q).clamp(min=0).sum())) < 2 * 2.0 ** -17 + 1e-5
    assert 0 <= int(vs.diag["draft_tokens"]) < V and int(accepted) in (0, 1) and 0 <= int(tokens) < V
    del vs, W, p, q
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
