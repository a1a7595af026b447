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


def _inputs(R, d, V, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = (torch.randn(V, d, generator=g, device="cuda") * 0.1).bfloat16()
    h = torch.randn(R, d, generator=g, device="cuda").bfloat16()
    return W, h, torch.randint(0, V, (R,), generator=g, device="cuda", dtype=torch.int32)


@pytest.mark.parametrize("d,V", [(64, 45057), (1024, 49152)])
def test_which_sums_a_workspace_gives(d, V):
    """With the size that the library names, those of one row tile; with room for whole tiles only, to the bit those of the two row tiles that
    a call of one more row takes (321: eight wavefronts too), and nothing is written past it."""
    W, h, labels = _inputs(321, d, V)

    def ce(R, nbytes=None):
        op = fb.HeadCrossEntropy(R, d, V)
        named = op.workspace.numel()
        room = torch.full((named + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        op.workspace = room[:named if nbytes is None else nbytes]
        out = op(h[:R], W, labels[:R])[0].clone()
        assert bool((room[op.workspace.numel():] == 0xA5).all())
        return out
    whole = -(-(320 * -(-V // 256) * 8) // 256) * 256 + 320 * 4
    one, two = ce(320), ce(320, whole)
    assert torch.equal(two, ce(321)[:320]) and torch.equal(ce(320, whole + 256), two)
    assert torch.equal(one[:257], ce(257)) and not torch.equal(one, two)


@pytest.mark.parametrize("R,V", [(257, 57344), (300, 50257), (320, 45057)])
def test_rows_that_do_not_count_labels_past_the_vocabulary_and_a_temperature(R, V):
    d, tau = 192, 0.7
    W, h, labels = _inputs(R, d, V, seed=R)
    labels[::7] = -100
    labels[3::50] = V - 1
    labels[5], labels[R - 1], labels[1] = V, 2**31 - 1, -2**31
    ce, loss = fb.HeadCrossEntropy(R, d, V)(h, W, labels, temperature=tau)
    scale = float(torch.tensor(1.0) / torch.tensor(tau))
    L = h.double() @ W.double().t().contiguous() * scale
    good = (labels >= 0) & (labels < V)
    want = torch.logsumexp(L, 1) - L.gather(1, labels.long().clamp(0, V - 1)[:, None])[:, 0]
    bound = 2 * shares._bound(h.double(), W.double(), d, scale).max(1).values + 2e-5
    assert bool(((ce - want).abs() <= bound)[good].all())
    assert bool((ce[labels < 0] == 0).all()) and bool(ce[labels >= V].isnan().all()) and bool(loss.isnan().all())


@pytest.mark.parametrize("first,last", [(640, 704), (16, 32), (1000, 3000), (50000, 50257)])
def test_tokens_of_logit_minus_infinity(first, last):
    """Tokens banned by an overflowing column of W, up to whole shares of them: no mass, no NaN, their neighbours keep theirs."""
    R, d, V = 300, 128, 50257
    W, h, labels = _inputs(R, d, V, seed=first)
    W[first:last, 0], h[:, 0] = -3e38, 8.0
    keep = torch.ones(V, dtype=torch.bool, device="cuda")
    keep[first:last] = False
    labels = torch.where((labels >= first) & (labels < last), torch.full_like(labels, first - 1), labels)
    ce, _ = fb.HeadCrossEntropy(R, d, V)(h, W, labels)
    L = h.double() @ W.double().t().contiguous()
    want = torch.logsumexp(L[:, keep], 1) - L.gather(1, labels.long()[:, None])[:, 0]
    bound = 2 * shares._bound(h.double(), W.double()[keep], d, 1.0).max(1).values + 2e-5
    assert bool(((ce - want).abs() <= bound).all())


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
