"""The three ways the round is finished (chunk masses of the rejected slot in a kernel of their own, of every slot, or
inside the final kernel for a small vocabulary) give the same round, on either side of the sizes where one takes over;
overlap and residual masses against float64."""
import pytest
import torch

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [1, 5, 255, 257, 1023, 4096, 4097, 9001])
@pytest.mark.parametrize("B,K,block,left", [(1, 4, 8, 6), (3, 8, 300, 280), (5, 16, 20, 7)])
def test_same_round_with_and_without_masses_of_every_slot(V, B, K, block, left):
    d = 64
    g = torch.Generator().manual_seed(V + B)
    W = torch.randn(V, d, generator=g).bfloat16().cuda()
    hd = torch.randn(B, K, d, generator=g)
    ht = (0.8 * hd + 0.6 * torch.randn(B, K, d, generator=g)).bfloat16().cuda()
    hd = hd.bfloat16().cuda()
    order = torch.rand(B, block, generator=g).argsort(1).argsort(1)
    mask = (order < left).to(torch.uint8).cuda()
    plain, full = fb.VerifyStep(B, K, block, d, V), fb.VerifyStep(B, K, block, d, V, diag=True, diag_logits=True)
    for step in range(4):
        for greedy in (False, True):
            got = []
            for vs in (plain, full):
                st = {"pass_mask": (1 - mask).contiguous(), "conf": torch.full((B, block), 0.5, device="cuda"),
                      "tokens_state": torch.zeros(B, block, dtype=torch.int32, device="cuda"),
                      "seq_pass": torch.zeros(B, dtype=torch.int32, device="cuda")}
                out = vs(hd, ht, W, 11, step=step, mask_in=mask, n_pass=2, greedy=greedy, **st)
                got.append([t.clone() for t in (*out, *st.values())])
            torch.cuda.synchronize()
            for x, y in zip(*got):
                assert torch.equal(x, y)
    window = min(K, left)
    L = full.diag["logits"].double()
    q, p = L.softmax(-1)[:, :, :window]
    # fp32 exponentials of logits below 64 in magnitude (relative error 2^-24 * 64 each) and sums of at most 9001 terms
    assert bool(((full.diag["alpha"][:, :window] - torch.minimum(p, q).sum(-1)).abs() < 2e-5).all())
    assert bool(((full.diag["resid_mass"][:, :window] - (p - q).clamp(min=0).sum(-1)).abs() < 2e-5).all())
    assert bool((full.diag["alpha"][:, window:] == 0).all())
