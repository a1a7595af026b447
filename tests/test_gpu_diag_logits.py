"""Diagnostic logits come from the kernel that computes every slot's masses where a call wants both, else from a copy: the same bits,
for rows that are and are not whole quads, a buffer that is only 4-byte aligned, slots past the window, and halves of a round."""
import pytest
import torch

from paper_2605_14305_amd import binding as fb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [3, 255, 256, 1021, 4095, 4100, 8190])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_same_logits_with_and_without_masses(V, offset):
    B, K, block, d = 2, 5, 8, 64
    g = torch.Generator(device="cuda").manual_seed(V)
    W = torch.randn(V, d, generator=g, device="cuda").bfloat16()
    hd, ht = (torch.randn(B, K, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    mask = torch.zeros(B, block, dtype=torch.uint8, device="cuda")
    mask[0, :3] = 1
    mask[1, 2:] = 1
    n = 2 * B * K * V

    def call(masses, *phases):
        vs = fb.VerifyStep(B, K, block, d, V, diag=True)
        buffer = torch.full((n + 8,), 7.5, device="cuda")
        vs.diag = dict(vs.diag if masses else {}, logits=buffer[offset:offset + n].view(2, B, K, V))
        for phase in phases:
            if phase == fb.FEF_PHASE_TARGET:
                buffer[:offset + n // 2] = 7.5  # the draft half's: not this call's to write
            vs(hd, ht, W, 3, mask_in=mask, phase=phase)
        torch.cuda.synchronize()
        return buffer

    whole = call(False, fb.FEF_PHASE_FUSED)
    assert bool((whole[:offset] == 7.5).all()) and bool((whole[offset + n:] == 7.5).all())
    assert torch.equal(whole, call(True, fb.FEF_PHASE_FUSED))
    half = call(False, fb.FEF_PHASE_DRAFT, fb.FEF_PHASE_TARGET)
    assert bool((half[:offset + n // 2] == 7.5).all())
    assert torch.equal(half, call(True, fb.FEF_PHASE_DRAFT, fb.FEF_PHASE_TARGET))
