"""The kernel that does the whole round of a toy model, against the separate kernels (which a call takes that asks for the masses of
every slot): the same bits in every output, at the edges of its range and one step past them."""
import pytest
import torch

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.gpu


def _run(B, K, d, V, alone, greedy=False, given=False, phases=(fb.FEF_PHASE_FUSED,), recorrupt=1.0):
    g = torch.Generator(device="cuda").manual_seed(B * 7 + K * 5 + d * 3 + V)
    W = torch.randn(V, d, generator=g, device="cuda")
    hd = torch.randn(B, K, d, generator=g, device="cuda") * (2.0 / d ** 0.5)
    ht = hd * 0.9 + torch.randn(B, K, d, generator=g, device="cuda") * (0.8 / d ** 0.5)
    block = K + 3
    left = torch.arange(B, device="cuda") % (block + 1)  # windows of every length, none among them
    mask = (torch.rand(B, block, generator=g, device="cuda").argsort(1).argsort(1) < left[:, None]).to(torch.uint8)
    state = dict(mask_in=mask, pass_mask=1 - mask, conf=torch.rand(B, block, generator=g, device="cuda"),
                 tokens_state=torch.randint(0, V, (B, block), generator=g, device="cuda", dtype=torch.int32),
                 seq_pass=torch.zeros(B, dtype=torch.int32, device="cuda"), seq_rounds=torch.zeros(B, dtype=torch.int32, device="cuda"))
    draft = torch.randint(0, V, (B, K), generator=g, device="cuda", dtype=torch.int32) if given else None
    vs = fb.VerifyStep(B, K, block, d, V, dtype="f32", diag=True)
    for t in vs.diag.values():
        t.zero_()
    if alone:
        vs.diag = {k: vs.diag[k] for k in ("draft_tokens", "lse", "conf_tok")}
    for step in range(2):
        for phase in phases:
            vs(hd, ht, W, 11, temperature=0.8, step=step, seq_base=5, pos_base=3, n_pass=3, draft_tokens=draft, greedy=greedy, phase=phase,
               recorrupt_prob=recorrupt, **state)
        state["mask_in"].copy_(vs.out_remask)
    torch.cuda.synchronize()
    return [vs.out_tokens, vs.out_accept_len, vs.out_remask, vs.diag["draft_tokens"], vs.diag["lse"], vs.diag["conf_tok"], *state.values()]


def _same(*args, **kw):
    for x, y in zip(_run(*args, True, **kw), _run(*args, False, **kw)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("V", [1, 2, 63, 64, 65, 130, 192, 255, 256, 257])
@pytest.mark.parametrize("d", [1, 31, 32, 36, 64, 97, 191, 192, 193])
def test_sizes(d, V):
    _same(3, 8, d, V)


@pytest.mark.parametrize("B,K", [(1, 1), (1, 4), (12, 7), (255, 8), (256, 8), (257, 8), (9, 9)])
@pytest.mark.parametrize("kw", [{}, dict(greedy=True), dict(given=True), dict(recorrupt=0.5)], ids=str)
def test_batches_and_options(B, K, kw):
    _same(B, K, 48, 200, **kw)


def test_halves_of_a_round():
    _same(4, 6, 64, 100, phases=(fb.FEF_PHASE_DRAFT, fb.FEF_PHASE_TARGET))
