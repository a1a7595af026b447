"""The kernel that does the whole round of a toy model, against the separate kernels (which a call takes that asks for the masses of
every slot): the same bits in every output, at the edges of its range and one step past them; and against the oracle."""
import numpy as np
import pytest
import torch

import parity
from oracle import fef_oracle as O
from paper_2605_14305_amd import binding as fb
from paper_2605_14305_amd import synth

pytestmark = pytest.mark.gpu


def _run(B, K, d, V, alone, greedy=False, given=False, phases=(fb.FEF_PHASE_FUSED,), recorrupt=1.0, block=None, without=(), **options):
    g = torch.Generator(device="cuda").manual_seed(B * 7 + K * 5 + d * 3 + V)
    W = torch.randn(V, d, generator=g, device="cuda")
    hd = torch.randn(B, K, d, generator=g, device="cuda") * (2.0 / d ** 0.5)
    ht = hd * 0.9 + torch.randn(B, K, d, generator=g, device="cuda") * (0.8 / d ** 0.5)
    block = K + 3 if block is None else block
    left = torch.arange(B, device="cuda") % (block + 1)  # windows of every length, none among them
    mask = (torch.rand(B, block, generator=g, device="cuda").argsort(1).argsort(1) < left[:, None]).to(torch.uint8)
    state = dict(mask_in=mask, pass_mask=1 - mask, conf=torch.rand(B, block, generator=g, device="cuda"),
                 tokens_state=torch.randint(0, V, (B, block), generator=g, device="cuda", dtype=torch.int32),
                 seq_pass=torch.zeros(B, dtype=torch.int32, device="cuda"), seq_rounds=torch.zeros(B, dtype=torch.int32, device="cuda"))
    state = {k: v for k, v in state.items() if k not in without}
    draft = torch.randint(0, V, (B, K), generator=g, device="cuda", dtype=torch.int32) if given else None
    vs = fb.VerifyStep(B, K, block, d, V, dtype="f32", diag=True)
    for t in vs.diag.values():
        t.zero_()
    if alone:
        vs.diag = {k: vs.diag[k] for k in ("draft_tokens", "lse", "conf_tok")}
    for step in range(2):
        for phase in phases:
            vs(hd, ht, W, 11, temperature=0.8, step=step, seq_base=5, pos_base=3, n_pass=3 if "seq_pass" in state else 0, draft_tokens=draft,
               greedy=greedy, phase=phase, recorrupt_prob=recorrupt, **options, **state)
        if "mask_in" in state:
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


STATE = ("mask_in", "pass_mask", "conf", "tokens_state", "seq_pass", "seq_rounds")


@pytest.mark.parametrize("without", [("mask_in",), ("pass_mask",), ("tokens_state",), ("seq_pass",), ("seq_rounds",), ("conf", "pass_mask"), STATE],
                         ids="+".join)
@pytest.mark.parametrize("block", [8, 64])
def test_state_that_is_not_given(without, block):
    for final_pass in (False, True):
        _same(5, 8, 64, 96, block=block, without=without, final_pass=final_pass)


@pytest.mark.parametrize("block", [9, 63, 64, 65, 255, 256, 257, 700, 4096])  # above 64 the uniforms are drawn another way, above 256 threads loop
@pytest.mark.parametrize("scope", [0, 1])
def test_blocks_and_what_is_re_masked(block, scope):
    for n_rm in (-1, 0, 1, block):
        _same(6, 7, 36, 130, block=block, lowconf_scope=scope, n_rm=n_rm)
        _same(6, 7, 36, 130, block=block, lowconf_scope=scope, n_rm=n_rm, without=("seq_pass",))


def test_halves_of_a_round():
    # the separate kernels, row range by row range, against the one kernel of a whole round
    for x, y in zip(_run(4, 6, 64, 100, True, phases=(fb.FEF_PHASE_DRAFT, fb.FEF_PHASE_TARGET)), _run(4, 6, 64, 100, True)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("B,K,block,d,V,kw", [
    (1, 4, 8, 64, 32, {}), (1, 4, 8, 64, 8, {}), (3, 8, 20, 100, 250, {}), (64, 8, 16, 64, 256, {}), (4, 5, 70, 192, 7, {}),
    (2, 7, 30, 48, 200, dict(greedy=True)), (5, 3, 3, 33, 256, dict(n_rm=2)), (5, 3, 3, 33, 64, dict(final_pass=True)),
    (4, 2, 5, 31, 100, dict(lowconf_scope=1)), (4, 2, 2, 64, 100, dict(recorrupt_prob=0.5))], ids=str)
def test_against_the_oracle(B, K, block, d, V, kw):
    total = dict(near_flipped=0, equal=0, rejected=0)
    W = synth.make_head(V, d, 3, "f32")
    for step in range(6):
        hd, ht = synth.make_hidden(B, K, d, 3, 0.6, 2.5 / (0.02 * np.sqrt(d)), "f32", 0, step)
        mask = np.zeros((B, block), np.uint8)  # windows of every length
        for b in range(B):
            mask[b, np.random.default_rng(100 * step + b).permutation(block)[:(b + step) % (block + 1)]] = 1
        conf = np.random.default_rng(step).uniform(0.1, 0.9, (B, block)).astype(np.float32)
        g_mask, g_conf, g_pass = (torch.from_numpy(x.copy()).cuda() for x in (mask, conf, 1 - mask))
        vs = fb.VerifyStep(B, K, block, d, V, dtype="f32", diag=True)
        vs.diag = {k: vs.diag[k] for k in ("draft_tokens", "lse", "conf_tok")}  # the masses would send it to the separate kernels
        out = vs(hd.cuda(), ht.cuda(), W.cuda(), 3, temperature=0.9, step=step, seq_base=2, pos_base=7, mask_in=g_mask, conf=g_conf,
                 pass_mask=g_pass, **kw)
        ref = O.verify_step(synth.to_f64(hd), synth.to_f64(ht), synth.to_f64(W), K, block, 3, temperature=0.9, step=step, seq_base=2, pos_base=7,
                            mask_in=mask, conf=conf, pass_mask=1 - mask, **kw)
        st = parity.compare(ref, *(t.cpu().numpy() for t in out), {k: t.cpu().numpy() for k, t in vs.diag.items()})
        total["near_flipped"] += st["near_flipped"]
        total["equal"] += st["equal"]
        total["rejected"] += int((ref.accept_len < ref.window).sum())
        if st["near_flipped"] == 0 and st["remask_skipped"] == 0:
            assert np.array_equal(g_pass.cpu().numpy(), ref.pass_mask)
            assert np.allclose(g_conf.cpu().numpy(), ref.conf, rtol=2e-4, atol=1e-12)  # as the parity tests have it
    assert total["near_flipped"] <= 1 and total["equal"] >= 6 * B - 1 and total["rejected"] > 0
