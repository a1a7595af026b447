"""Cross-entropy of 257 to 320 rows in one row tile (csrc/head_loss.hip) against a float64 product: edges of its rows and shares."""
import pytest
import torch

from paper_2605_14305_amd import binding as fb
import test_gpu_shares as shares

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [45057, 49152, 50257, 57344])
@pytest.mark.parametrize("d", [64, 128, 192, 1024])
def test_against_a_float64_product(d, V):
    for R in (257, 272, 303, 304) + ((305, 320) if V <= 49152 else ()):
        shares._check_loss(R, d, V)


def test_a_workspace_with_room_for_whole_tiles_only():
    """What two row tiles leave fits: the call takes them, as before there was another way."""
    R, d, V = 300, 128, 50257
    g = torch.Generator(device="cuda").manual_seed(1)
    W = (torch.randn(V, d, generator=g, device="cuda") * 0.1).bfloat16()
    h = torch.randn(R, d, generator=g, device="cuda").bfloat16()
    labels = torch.randint(0, V, (R,), generator=g, device="cuda", dtype=torch.int32)
    op = fb.HeadCrossEntropy(R, d, V)
    ce = op(h, W, labels)[0].clone()
    whole, workspace = -(-(R * -(-V // 256) * 8) // 256) * 256 + -(-R * 4 // 256) * 256, op.workspace
    assert whole < workspace.numel()
    op.workspace = workspace[:whole]
    # log-sum-exps of the same logits by two orders of 50257 terms
    assert bool(((op(h, W, labels)[0] - ce).abs() <= 4e-5).all())
    op.workspace = workspace[:whole - 256]
    with pytest.raises(fb.FefError) as e:
        op(h, W, labels)
    assert e.value.status == fb.FEF_ERR_WORKSPACE
