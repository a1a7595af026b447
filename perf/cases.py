"""Performance cases of the verify-step library: what a decoding or training program has it do.

A case is one call (or one draft call followed by its target call) through the public binding with the
head W and the hidden states resident on the GPU.  Inputs are what the path meets in earnest: each slot's
hidden state points at a predicted token of its own on top of noise over the whole vocabulary, so the laws are
peaked (the predicted token holds most of the mass) with a long tail, and draft and target agree on that token
in nine of ten slots, which gives the acceptance rates a trained draft shows.
"""
import math

import numpy as np
import torch

from paper_2605_14305_amd import binding as fb

_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest call: a toy model's fp32 head; latency and launches are all it costs
        dict(name="tiny_f32", kind="round", B=1, K=4, block=8, d=64, V=32, dtype="f32", tau=1.0),
        # fp32 head of a small model with everything written out: what one runs to check numerics
        dict(name="f32_logits", kind="logits", B=2, K=8, block=32, d=1024, V=32000, dtype="f32", tau=1.0),
        # interactive decoding of one sequence with an 8B model's head (4096 x 126464), window of 8
        dict(name="llada_b1", kind="round", B=1, K=8, block=32, d=4096, V=126464, dtype="bf16", tau=1.0),
        # the same in the method's own call order: draft call, model forward, target call
        dict(name="llada_b1_split", kind="split", B=1, K=8, block=32, d=4096, V=126464, dtype="bf16", tau=1.0),
        # one sequence, 7B model with a larger vocabulary, the paper's window of 16
        dict(name="dream_b1", kind="round", B=1, K=16, block=64, d=3584, V=151936, dtype="bf16", tau=1.0),
        # greedy decoding of two sequences with a small model's head
        dict(name="small_greedy", kind="greedy", B=2, K=8, block=32, d=1536, V=32000, dtype="bf16", tau=1.0),
        # a few sequences in flight, nothing a round number
        dict(name="ragged_b5", kind="round", B=5, K=11, block=37, d=2560, V=100003, dtype="bf16", tau=0.8),
        # batched serving
        dict(name="llada_b16", kind="round", B=16, K=8, block=32, d=4096, V=126464, dtype="bf16", tau=1.0),
        # acceptance sweep at scale: 64 sequences, window of 16, overlap and residual mass of every slot
        dict(name="sweep_b64", kind="diag", B=64, K=16, block=32, d=4096, V=126464, dtype="bf16", tau=1.0),
        # the baseline decoder the speed-ups are relative to: two tokens of a 32-position block per step
        dict(name="topn_b1", kind="topn", B=1, K=32, block=32, d=4096, V=126464, dtype="bf16", tau=1.0),
        # token-level training loss of 2048 position-conditioned rows
        dict(name="ce_2048", kind="ce", R=2048, d=4096, V=126464, dtype="bf16", tau=1.0),
        # the same for a small model and a ragged batch
        dict(name="ce_ragged", kind="ce", R=300, d=2048, V=50257, dtype="bf16", tau=1.0),
    ]


_LARGEST_FLOPS = 2.0 * 2048 * 126464 * 4096


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    while True:
        kind = rng.choice(["round", "round", "round", "split", "greedy", "diag", "topn", "ce", "ce", "logits", "tiny"])
        tau = rng.choice([0.5, 0.8, 1.0, 1.0])
        if kind in ("tiny", "logits"):  # fp32 heads: toy and small models
            d, V = (log(16, 128), log(8, 512)) if kind == "tiny" else (log(128, 1024), log(2000, 32000))
            K = rng.randint(2, 8)
            return dict(kind="round" if kind == "tiny" else "logits", B=rng.randint(1, 3), K=K, block=K + rng.randint(2, 25),
                        d=d, V=V, dtype="f32", tau=tau)
        d = rng.choice([512, 1024, 1536, 2048, 2560, 3072, 3584, 4096, 64 * rng.randint(8, 64)])
        V = rng.choice([126464, 151936, log(8000, 152000), log(8000, 152000)])
        if kind == "ce":
            c = dict(kind="ce", R=log(16, 2048), d=d, V=V, dtype="bf16", tau=1.0)
            rows = c["R"]
        else:
            K = rng.choice([4, 8, 16, rng.randint(1, 32)])
            c = dict(kind=kind, B=log(1, 64), K=K, block=K + rng.randint(4, 48), d=d, V=V, dtype="bf16", tau=tau)
            rows = 2 * c["B"] * K
        # diagnostics of every slot read all logits again: the largest listed case has them too
        if 2.0 * rows * d * V <= _LARGEST_FLOPS:
            return c


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + 12345) & 0x7FFFFFFFFFFFFFFF)
    return g


def _head(c, g):
    W = torch.empty(c["V"], c["d"], dtype=_DTYPE[c["dtype"]], device="cuda")
    for v in range(0, c["V"], 16384):  # in pieces: no fp32 copy of the whole head
        n = min(16384, c["V"] - v)
        W[v:v + n] = torch.randn(n, c["d"], generator=g, device="cuda").mul_(0.02)
    return W


def _hidden(c, W, tokens, noise):
    """Rows whose scaled logits have a standard deviation of about 2 and whose token `tokens` stands
    out by enough to hold most of the mass: ln V + 2 is the log-sum-exp of the noise."""
    std = 2.0
    lift = math.log(max(c["V"], 2)) + std * std / 2 + 5.0
    w = W[tokens].float()
    h = noise * (std / (0.02 * math.sqrt(c["d"]))) + w * (lift / w.square().sum(-1, keepdim=True))
    return (h * c["tau"]).to(_DTYPE[c["dtype"]])


def _inputs(c, seed):
    """Everything a program has in hand before the call, with the state that the call updates."""
    g = _gen(seed)
    d, V = c["d"], c["V"]
    x = {"W": _head(c, g)}
    if c["kind"] == "ce":
        R = c["R"]
        labels = torch.randint(0, V, (R,), generator=g, device="cuda")
        right = torch.rand(R, generator=g, device="cuda") < 0.7  # rows whose label the model already predicts
        guess = torch.where(right, labels, torch.randint(0, V, (R,), generator=g, device="cuda"))
        x["h"] = _hidden(c, x["W"], guess, torch.randn(R, d, generator=g, device="cuda"))
        skip = torch.rand(R, generator=g, device="cuda") < 0.1   # positions that do not count
        x["labels"] = torch.where(skip, torch.full_like(labels, -100), labels).to(torch.int32)
        return x
    B, K, block = c["B"], c["K"], c["block"]
    target = torch.randint(0, V, (B, K), generator=g, device="cuda")
    agree = torch.rand(B, K, generator=g, device="cuda") < 0.9
    draft = torch.where(agree, target, torch.randint(0, V, (B, K), generator=g, device="cuda"))
    nd = torch.randn(B, K, d, generator=g, device="cuda")
    nt = 0.9 * nd + math.sqrt(1 - 0.81) * torch.randn(B, K, d, generator=g, device="cuda")
    x["hd"] = _hidden(c, x["W"], draft, nd)
    x["ht"] = _hidden(c, x["W"], target, nt)
    # a block part of the way through: more positions unresolved than the window takes (all of them where
    # the window is the block), the others committed earlier with their confidences
    left = block if K == block else max(K + 1, (3 * block) // 4)
    order = torch.rand(B, block, generator=g, device="cuda").argsort(1).argsort(1)
    mask = (order < left).to(torch.uint8)
    done = mask == 0
    x["mask"] = mask
    x["pass_mask"] = done.to(torch.uint8)
    x["conf"] = torch.where(done, 0.3 + 0.7 * torch.rand(B, block, generator=g, device="cuda"), torch.zeros((), device="cuda"))
    x["tokens"] = torch.where(done, torch.randint(0, V, (B, block), generator=g, device="cuda"),
                              torch.full((), -1, device="cuda")).to(torch.int32)
    return x


def prepare(case, seed):
    s = _inputs(case, seed)
    s["c"], s["seed"] = case, int(seed)
    if case["kind"] == "ce":
        s["op"] = fb.HeadCrossEntropy(case["R"], case["d"], case["V"], dtype=case["dtype"])
    else:
        s["op"] = fb.VerifyStep(case["B"], case["K"], case["block"], case["d"], case["V"], dtype=case["dtype"],
                                diag=case["kind"] in ("diag", "logits"), diag_logits=case["kind"] == "logits")
    return s


_STEP = 3  # index of the round, the same in every pass


def run(s):
    c, op, seed = s["c"], s["op"], s["seed"]
    if c["kind"] == "ce":
        ce, loss = op(s["h"], s["W"], s["labels"], temperature=c["tau"])
        return {"ce": ce, "loss": loss}
    if c["kind"] == "topn":
        tok, n, rem = fb.topn_step(op, s["hd"], s["W"], seed, 2, temperature=c["tau"], step=_STEP, mask_in=s["mask"],
                                   conf=s["conf"], tokens_state=s["tokens"])
        return {"tokens": tok, "committed": n, "remask": rem, "conf": s["conf"], "state": s["tokens"]}
    kw = dict(temperature=c["tau"], step=_STEP, mask_in=s["mask"], pass_mask=s["pass_mask"], conf=s["conf"],
              tokens_state=s["tokens"], greedy=c["kind"] == "greedy")
    if c["kind"] == "split":
        op(s["hd"], None, s["W"], seed, phase=fb.FEF_PHASE_DRAFT, **kw)
        tok, acc, rem = op(None, s["ht"], s["W"], seed, phase=fb.FEF_PHASE_TARGET, **kw)
    else:
        tok, acc, rem = op(s["hd"], s["ht"], s["W"], seed, **kw)
    out = {"tokens": tok, "accepted": acc, "remask": rem, "conf": s["conf"], "pass": s["pass_mask"], "state": s["tokens"]}
    if op.diag:
        out.update(op.diag)
    return out


def work(case):
    """W and the hidden states read once (W once in each half of a split round: the target half waits for a
    model forward that needs the draft tokens), the outputs written once.  The logits count only where they
    are an output."""
    c = case
    rows = c["R"] if c["kind"] == "ce" else c["B"] * c["K"] * (1 if c["kind"] == "topn" else 2)
    esz = 2 if c["dtype"] == "bf16" else 4
    nbytes = c["V"] * c["d"] * esz * (2 if c["kind"] == "split" else 1) + rows * c["d"] * esz
    if c["kind"] == "ce":
        nbytes += 8 * rows
    else:
        nbytes += c["B"] * c["block"] * (2 + 2 + 8 + 8) + c["B"] * c["K"] * 4 + c["B"] * 4
        nbytes += c["B"] * c["K"] * 4 * 6 if c["kind"] in ("diag", "logits") else 0
        nbytes += rows * c["V"] * 4 if c["kind"] == "logits" else 0
    return {"bytes": nbytes, "flops": 2 * rows * c["d"] * c["V"]}


def tolerance(case):
    # 32-bit sums and softmax throughout.  A draw from the tail of a law may land on the token next to it
    # (the prefix sums of two correct implementations differ by some 1e-7, the tail's tokens are no heavier).
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.01}


# ------------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------------
def _uniform(seed, position, step, sequence, stream):
    """Philox4x32-10 (Salmon et al., SC'11), first output word, top 23 bits, as the library documents its draws."""
    m32 = 0xFFFFFFFF
    k0, k1 = seed & m32, (seed >> 32) & m32
    c = [position & m32, step & m32, sequence & m32, stream]
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
        p0, p1 = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(p1 >> 32) ^ c[1] ^ k0, p1 & m32, (p0 >> 32) ^ c[3] ^ k1, p0 & m32]
    return ((c[0] >> 9) + 0.5) * 2.0 ** -23


def _logits(h, W, tau):
    h = h.reshape(-1, h.shape[-1]).double()
    out = torch.empty(h.shape[0], W.shape[0], dtype=torch.float64, device=W.device)
    for v in range(0, W.shape[0], 16384):
        out[:, v:v + 16384] = h @ W[v:v + 16384].double().t().contiguous()
    return out.div_(tau)


def _pick(mass, u):
    """First index whose prefix sum reaches u times the total."""
    cum = mass.cumsum(0)
    return min(int(torch.searchsorted(cum, u * cum[-1])), mass.numel() - 1)


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    if c["kind"] == "ce":
        L = _logits(x["h"], x["W"], c["tau"])
        lab = x["labels"].long()
        ce = torch.logsumexp(L, 1) - L.gather(1, lab.clamp(min=0)[:, None])[:, 0]
        ce = torch.where(lab >= 0, ce, torch.zeros_like(ce))
        return {"ce": ce, "loss": ce.sum()[None]}
    B, K, block, seed = c["B"], c["K"], c["block"], int(seed)
    Lq = _logits(x["hd"], x["W"], c["tau"])
    lse_q = torch.logsumexp(Lq, 1)
    slots = [[i for i, m in enumerate(row) if m][:K] for row in x["mask"].cpu().tolist()]
    conf = x["conf"].double()

    def drawn(row, b, pos):
        if c["kind"] == "greedy":
            return int(Lq[row].argmax())
        return _pick((Lq[row] - lse_q[row]).exp(), _uniform(seed, pos, _STEP, b, 0))

    if c["kind"] == "topn":
        for b in range(B):
            p = []
            for m, pos in enumerate(slots[b]):
                t = drawn(b * K + m, b, pos)
                p.append((float((Lq[b * K + m, t] - lse_q[b * K + m]).exp()), pos))
            for q, pos in sorted(p, key=lambda e: (-e[0], e[1]))[:2]:
                conf[b, pos] = q
        return {"tokens": None, "committed": None, "remask": None, "conf": conf, "state": None}
    Lp = _logits(x["ht"], x["W"], c["tau"])
    lse_p = torch.logsumexp(Lp, 1)
    conf_tok = np.zeros((B, K))
    for b in range(B):
        for m, pos in enumerate(slots[b]):
            r = b * K + m
            t = drawn(r, b, pos)
            lp, lq = float(Lp[r, t] - lse_p[r]), float(Lq[r, t] - lse_q[r])
            if c["kind"] == "greedy":
                best = int(Lp[r].argmax())
                ok, other = t == best, best
            else:
                ok, other = _uniform(seed, pos, _STEP, b, 1) <= math.exp(min(0.0, lp - lq)), None
            if not ok:
                if other is None:
                    rest = ((Lp[r] - lse_p[r]).exp() - (Lq[r] - lse_q[r]).exp()).clamp(min=0)
                    other = _pick(rest, _uniform(seed, pos, _STEP, b, 2))
                lp = float(Lp[r, other] - lse_p[r])
            conf_tok[b, m] = math.exp(lp)
            conf[b, pos] = conf_tok[b, m]
            if not ok:
                break
    out = {"tokens": None, "accepted": None, "remask": None, "conf": conf, "pass": None, "state": None}
    if c["kind"] in ("diag", "logits"):
        alpha = torch.empty(B * K, dtype=torch.float64, device="cuda")
        resid = torch.empty_like(alpha)
        for r in range(B * K):
            p, q = (Lp[r] - lse_p[r]).exp(), (Lq[r] - lse_q[r]).exp()
            alpha[r], resid[r] = torch.minimum(p, q).sum(), (p - q).clamp(min=0).sum()
        out.update(draft_tokens=None, alpha=alpha.view(B, K), resid_mass=resid.view(B, K),
                   lse=torch.stack([lse_q, lse_p]).view(2, B, K), conf_tok=torch.from_numpy(conf_tok).cuda())
        if c["kind"] == "logits":
            out["logits"] = torch.stack([Lq, Lp]).view(2, B, K, c["V"])
    return out
