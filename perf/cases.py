"""The workloads this framework's speed is judged on: whole calls of the training step, as a training or
validation program makes them through Session and Trainer.

A case names a model, a form (how the sentences go through the library), the token budget and number of its
sub-batches and the length distribution of its sentences.  Sentence lengths follow from the case alone, so that
its work is fixed; weights, token ids and dropout streams follow from the seed.

Forms
  update    Trainer.step over padded sub-batches one by one (forward + loss, backward, accumulate for each), then
            overflow check and Adam
  group     the same update with all sub-batches stacked row-wise into one pass, padding kept
  packed    the same update with all sentences back to back in one pass, no padding
  validate  forward pass and loss without dropout over one packed pass, no gradient
"""
from __future__ import annotations

import math
import weakref

import numpy as np
import torch

from paper_1806_00187_amd.session import Session, Trainer

PAD, BOS = 1, 2
MAX_LEN = 256

MODELS = {
    "tiny": dict(enc_layers=2, dec_layers=2, d_model=64, n_heads=4, d_ff=256, vocab=1000, dropout=0.1),
    "small": dict(enc_layers=2, dec_layers=2, d_model=256, n_heads=4, d_ff=1024, vocab=2056, dropout=0.1),
    "base": dict(enc_layers=6, dec_layers=6, d_model=512, n_heads=8, d_ff=2048, vocab=32768, dropout=0.1),
    "big": dict(enc_layers=6, dec_layers=6, d_model=1024, n_heads=16, d_ff=4096, vocab=32768, dropout=0.3),
    "big40k": dict(enc_layers=6, dec_layers=6, d_model=1024, n_heads=16, d_ff=4096, vocab=40000, dropout=0.3),
}


def _case(name, model, form, sub_batches, budget, mean, sigma, pick, len_seed):
    return dict(name=name, model=model, form=form, sub_batches=sub_batches, budget=budget, mean=mean, sigma=sigma, pick=pick,
                len_seed=len_seed)


def listed():
    return [
        # the two-layer model on a sub-batch of about 130 tokens: a unit test's or tutorial's step, bound by launches
        _case("tiny_step", "tiny", "update", 1, 136, 16.0, 0.2, "median", 1001),
        # a 256-wide model on two ragged sub-batches of odd sizes, accumulated one by one
        _case("small_two_ragged", "small", "update", 2, 1531, 21.0, 0.6, "random", 1006),
        # Transformer-base on one sub-batch of the usual 3584-token budget, the ordinary single-GPU step
        _case("base_step", "base", "update", 1, 3584, 27.0, 0.6, "median", 1002),
        # the same budget filled with the longest sentences of the population (up to 256 positions): long attention
        _case("base_longest", "base", "update", 1, 3584, 27.0, 0.6, "longest", 1002),
        # four sub-batches of different shapes, padding kept, as one pass
        _case("base_group4", "base", "group", 4, 3584, 27.0, 0.6, "spread", 1002),
        # validation loss over eight sub-batches' worth of sentences, forward only
        _case("base_validate", "base", "validate", 8, 3584, 27.0, 0.6, "spread", 1002),
        # Transformer-big on a small batch (fine-tuning, the remainder of an epoch): few rows, many weights
        _case("big_few_tokens", "big", "update", 1, 448, 27.0, 0.6, "median", 1003),
        # Transformer-big with one 3584-token sub-batch per update
        _case("big_step", "big", "update", 1, 3584, 27.0, 0.6, "median", 1003),
        # gradient accumulation in the method's literal order: four sub-batches one after another
        _case("big_accum4_in_order", "big", "update", 4, 3584, 27.0, 0.6, "random", 1004),
        # V = 40000, longer sentences, four 5120-token sub-batches packed into one pass
        _case("big40k_accum4_packed", "big40k", "packed", 4, 5120, 35.0, 0.7, "random", 1005),
        # the sixteen sub-batches of a large-batch update packed into one pass
        _case("big_accum16_packed", "big", "packed", 16, 3584, 27.0, 0.6, "random", 1004),
    ]


def draw(rng):
    model = rng.choice(["tiny", "small", "base", "base", "big", "big", "big40k"])
    form = rng.choice(["update", "update", "group", "packed", "packed", "validate"])
    budget = int(round(math.exp(rng.uniform(math.log(100), math.log(5120)))))
    # at most what the largest listed case holds: 16 sub-batches of 3584 tokens at V = 32768
    most = {"big40k": 44000, "big": 56000}.get(model, 57344) // budget
    if form == "update":
        most = min(most, 4)
    sub_batches = rng.randint(1, max(1, min(16, most)))
    mean = math.exp(rng.uniform(math.log(8), math.log(90)))
    sigma = rng.uniform(0.2, 0.7)
    c = _case("", model, form, sub_batches, budget, round(mean, 2), round(sigma, 2), rng.choice(["median", "random", "spread", "longest"]),
              rng.randrange(1 << 20))
    del c["name"]
    return c


def _lengths(case):
    """Sub-batches as lists of (source length, target length): a population of sentences with lognormal target lengths
    and sources within 20 % of them, sorted by length, cut into sub-batches of sentences x longest <= budget; `pick`
    says which of those the case takes."""
    rng = np.random.default_rng(case["len_seed"])
    budget, k = case["budget"], case["sub_batches"]
    longest = min(MAX_LEN, budget)
    n = 40 * k * max(8, budget // max(1, int(case["mean"])))
    n = min(n, 100_000)
    tgt = np.clip(np.rint(rng.lognormal(math.log(case["mean"]) - 0.5 * case["sigma"] ** 2, case["sigma"], size=n)), 1, longest).astype(int)
    src = np.clip(np.rint(tgt * (1.0 + rng.uniform(-0.2, 0.2, size=n))), 1, longest).astype(int)
    order = np.lexsort((src, tgt))
    cuts, cur, widest = [], [], 0
    for i in order:
        m = max(widest, src[i], tgt[i])
        if cur and (len(cur) + 1) * m > budget:
            cuts.append(cur)
            cur, m = [], max(src[i], tgt[i])
        cur.append((int(src[i]), int(tgt[i])))
        widest = m
    cuts.append(cur)
    nb = len(cuts)
    if case["pick"] == "median":
        at = [min(nb - 1, max(0, nb // 2 - k // 2) + j) for j in range(k)]
    elif case["pick"] == "longest":
        at = [max(0, nb - 2 - j) for j in range(k)]      # (the very last one may be a small remainder)
    elif case["pick"] == "spread":
        at = [int(round(q * (nb - 1))) for q in np.linspace(0.05, 0.95, k)]
    else:
        at = [int(i) for i in rng.integers(0, nb, size=k)]
    return [cuts[i] for i in at]


def _sub_batch(lengths, vocab, cdf, rng):
    """Right-padded ids of one sub-batch: Zipf-distributed words, the decoder input shifted right behind BOS."""
    B, S, T = len(lengths), max(s for s, _ in lengths), max(t for _, t in lengths)
    word = lambda shape: (np.minimum(np.searchsorted(cdf, rng.random(shape)), vocab - 5) + 4).astype(np.int32)
    src, out = word((B, S)), word((B, T))
    for b, (s, t) in enumerate(lengths):
        src[b, s:] = PAD
        out[b, t:] = PAD
    tin = np.full((B, T), PAD, dtype=np.int32)
    tin[:, 0] = BOS
    tin[:, 1:] = np.where(out[:, 1:] == PAD, PAD, out[:, :-1])
    return {"src": src, "tgt_in": tin, "tgt_out": out}


def _weights(model, layout, total, seed):
    """Xavier-uniform matrices, zero biases and shifts, unit gains, rounded to fp16: name -> array."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    flat = torch.empty(total, dtype=torch.float16, device="cuda").uniform_(-1.0, 1.0, generator=g)
    d = model["d_model"]
    for name, (off, rows, cols) in layout.items():
        t = flat[off:off + rows * cols]
        if rows > 1:
            fan_out = d if name.endswith(("wqkv", "wkv")) else rows       # stacks of d x d matrices
            t.mul_(math.sqrt(6.0 / (fan_out + cols)))
        else:
            t.fill_(1.0 if name.endswith(".g") else 0.0)
    host = flat.cpu().numpy()
    return {name: host[off:off + rows * cols] for name, (off, rows, cols) in layout.items()}


def _layout(model):
    """name -> (offset, rows, cols) of the flat parameter vector, asked of the library."""
    import paper_1806_00187_amd as nmt
    cfg = {k: v for k, v in model.items()}
    ctx = nmt.nmt_create(**cfg, pad_id=PAD, ln_eps=1e-5, label_smoothing=0.1, max_sentences=1, max_len=MAX_LEN)
    out = {}
    for i in range(nmt.nmt_param_tensors(ctx)):
        name, off, rows, cols = nmt.nmt_param_info(ctx, i)
        out[name] = (off, rows, cols)
    total = nmt.nmt_param_count(ctx)
    nmt.nmt_destroy(ctx)
    return out, total


class State:
    """What a training program holds between updates; the session is closed with it."""

    def __init__(self, case, seed):
        model = MODELS[case["model"]]
        lengths = _lengths(case)
        layout, total = _layout(model)
        self.validate = case["form"] == "validate"
        self.session = Session(model, _weights(model, layout, total, seed), max_sentences=max(len(b) for b in lengths), max_len=MAX_LEN,
                               seed=seed, optimizer=not self.validate)
        weakref.finalize(self, self.session.close)
        w = 1.0 / np.power(np.arange(1, model["vocab"] - 3, dtype=np.float64), 1.1)
        cdf, rng = np.cumsum(w) / w.sum(), np.random.default_rng(seed)
        batches = [_sub_batch(b, model["vocab"], cdf, rng) for b in lengths]
        self.n_tok = sum(t for b in lengths for _, t in b)
        s = self.session
        shapes = [(b["src"].shape[0], b["src"].shape[1], b["tgt_in"].shape[1], j) for j, b in enumerate(batches)]
        if case["form"] == "update":
            self.batches = [s.to_device(b) for b in batches]
            for shape in shapes:
                s.reserve(*shape[:3])
        else:
            self.batches = s.group([s.to_device(b) for b in batches], len(batches)) if case["form"] == "group" else s.pack(batches)
            s.reserve(shapes)
        # a loss scale the first updates from these weights are clear of overflow at (the scaler settles at 32)
        self.trainer = None if self.validate else Trainer(s, peak_lr=5e-4, init_scale=16.0)


def prepare(case, seed):
    return State(case, seed)


def run(state):
    s = state.session
    if state.validate:
        s.forward_loss(state.batches[0], 1.0, 0, training=False)
        return {"loss": s.loss_sum, "tokens": s.ntok, "decoder_output": s.activation("dec%d.out" % (s.model["dec_layers"] - 1))}
    loss, tokens, skipped = state.trainer.step(state.batches, n_tok=state.n_tok)
    return {"loss": loss, "tokens": tokens, "skipped": skipped, "gradient": s.g16, "accumulated": s.acc, "master": s.master, "adam_m": s.m,
            "adam_v": s.v, "weights": s.w16}


def work(case):
    m = MODELS[case["model"]]
    d, F, V, Le, Ld = m["d_model"], m["d_ff"], m["vocab"], m["enc_layers"], m["dec_layers"]
    lengths = np.array([p for b in _lengths(case) for p in b], dtype=np.float64)
    s, t = lengths[:, 0], lengths[:, 1]
    # matrix products over real positions (causal attention counts half a square); a backward pass is two forwards
    fwd = (Le * (s * (8 * d * d + 4 * d * F) + 4 * s * s * d)
           + Ld * (t * (12 * d * d + 4 * d * F) + s * 4 * d * d + 2 * t * t * d + 4 * t * s * d) + 2 * t * d * V).sum()
    P = V * d + Le * (4 * d * d + 2 * d * F + 9 * d + F) + Ld * (8 * d * d + 2 * d * F + 15 * d + F)
    ids = 4 * (s + 2 * t).sum()
    if case["form"] == "validate":
        return {"bytes": float(2 * P + ids + 2 * t.sum() * d), "flops": float(fwd)}
    # per parameter: fp16 weight, master weight and both moments in; gradient, accumulator, master, moments, weight out
    return {"bytes": float((2 + 12 + 2 + 4 + 12 + 2) * P + ids), "flops": float(3 * fwd)}


def tolerance(case):
    # Four times what the path differs from itself by when the hidden units of every feed-forward layer are permuted (the
    # same model, its contractions summed in another order).  Gradients of few tokens differ most, because a ReLU gate at
    # zero moves a larger share of them: 0.0051 (largest single value 0.67) at 305 tokens, 0.0024 (0.16) at 1673, 0.0009
    # (0.055) at 17700; the last decoder block's output 0.0007 (0.0044).
    if case["form"] == "validate":
        return {"rel": 0.003, "max": 0.02}
    if sum(t for b in _lengths(case) for _, t in b) < 1500 * case["sub_batches"]:
        return {"rel": 0.02, "max": 0.99}
    return {"rel": 0.01, "max": 0.65}
