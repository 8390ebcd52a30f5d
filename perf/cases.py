"""The work that a user of this package has it do, as a list of timed cases: training steps in both precisions
(forward and backward, with and without the update), the forward-only evaluation, greedy decoding and beam search, from
one sentence to full batches.

Shapes are the workloads of paper_1802_07170_amd/inputs.py where it has one, and generic otherwise.  Parameters come
from the library's own generator at +-0.05: the network is then in the range where its gradient is well conditioned, as
a network in training is (at +-0.1 and hidden size 1024 the recurrences amplify the rounding of any 16-bit operand).
Decoders get what training adds to that (see _as_trained)."""
from __future__ import annotations

import math

import torch

from paper_1802_07170_amd import binding, inputs as I

BEAM, LENGTH_PENALTY = 10, 0.6                 # the paper's search settings
DROPOUT, SMOOTHING, RATE = 0.2, 0.1, 0.1       # its regularisation; a learning rate from within its decay schedule
SCALE = 0.05                                   # parameters: uniform[-SCALE, SCALE)
WIDTHS = [64, 128, 256, 512, 1024]             # the usual hidden sizes, drawn as often as odd ones


def _workload(name):
    c = I.CONFIGS[name]
    return dict(vocab=c["src_vocab"], emb=c["emb"], hidden=c["hidden"], layers=c["layers"], precision=c["precision"],
                batch=c["batch"], lo=c["len_range"][0], hi=c["len_range"][1])


def listed():
    medium = _workload("medium")
    return [
        # the quick start: one blocking fp32 step of a toy network; nothing but launches and latency
        dict(name="tiny_step", kind="step", **_workload("tiny")),
        # a mid-sized network trained in full precision, sentences of 10 to 50 tokens
        dict(name="small_step", kind="async", **_workload("small")),
        # the 4-layer, 1024-wide network of the benchmark's headline figure
        dict(name="medium_step", kind="async", **medium),
        # the same network with the larger vocabulary, twice the batch and longer sentences
        dict(name="large_step", kind="async", **_workload("large")),
        # long sentences: every decoder position attends to 120 source positions
        dict(name="attn_step", kind="async", **_workload("attn")),
        # the training loop's iteration as the paper trains: a new dropout mask, the step, the update
        dict(name="paper_update", kind="update", **_workload("paper_512x2")),
        # a step with no round number anywhere: widths that are no multiple of 32, very uneven sentences
        dict(name="ragged_step", kind="async", vocab=9064, emb=200, hidden=336, layers=3, precision=1, batch=23, lo=3, hi=37),
        # the development-set cross-entropy that the learning-rate rule watches
        dict(name="medium_eval", kind="eval", **medium),
        # translating a batch with the best token of every step
        dict(name="medium_greedy", kind="greedy", **medium),
        # translating one sentence as it arrives, in full precision
        dict(name="single_greedy", kind="greedy", **dict(_workload("small"), batch=1, lo=25, hi=25)),
        # translating a batch with the paper's beam search: 640 decoder rows
        dict(name="medium_beam", kind="beam", **medium),
        # beam search over one sentence as it arrives
        dict(name="single_beam", kind="beam", **dict(medium, batch=1, lo=25, hi=25)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind of call, hidden sizes 64 to 1024, 1 to 4 layers, 1 to 128 sentences of up to 120 tokens,
    vocabularies of 1000 to 50000.  The batch is halved until the case costs no more than the large step; full precision
    counts 16-fold, as its matrix cores are that much slower."""
    kind = rng.choice(["step", "async", "async", "async", "update", "eval", "greedy", "beam"])
    hidden = rng.choice([rng.choice(WIDTHS), 16 * _log_int(rng, 4, 64)])
    hi = _log_int(rng, 6, 120)
    case = dict(kind=kind, vocab=8 * _log_int(rng, 125, 6250), emb=rng.choice([hidden, hidden, 8 * _log_int(rng, 8, 128)]), hidden=hidden,
                layers=rng.randint(1, 4), precision=rng.choice([0, 1, 1]), batch=_log_int(rng, 1, 64 if kind == "beam" else 128),
                lo=rng.randint(max(1, hi // 5), hi), hi=hi)
    budget = 0.8 * work(dict(_workload("large"), kind="async"))["flops"] / (1 if case["precision"] else 16)
    while case["batch"] > 1 and work(case)["flops"] > budget:
        case["batch"] //= 2
    return case


def _model(case):
    return dict(src_vocab=case["vocab"], tgt_vocab=case["vocab"], emb=case["emb"], hidden=case["hidden"], layers=case["layers"])


def _as_trained(trainer, case, seed):
    """Embeddings large enough that the tokens drive the decoder's state, so that a translation does not repeat one
    token.  For 16-bit operands also output biases that carry the log frequency of every token, as trained ones do: the
    best token is then ahead by more than the rounding of the operands, and which it is does not hang on a near tie."""
    place = {name: (offset, rows * cols) for name, rows, cols, offset in trainer.param_table()}
    for name in ("E_src", "E_tgt"):
        offset, n = place[name]
        trainer.params[offset:offset + n] *= 1.0 / SCALE
    if case["precision"]:
        words = case["vocab"] - 4
        generator = torch.Generator(device=trainer.device).manual_seed(seed)
        token = torch.randperm(words, generator=generator, device=trainer.device) + 4
        offset, n = place["B_o"]
        bias = trainer.params[offset:offset + n]
        bias.fill_(-1.1 * math.log(case["vocab"]))
        bias[token] = -1.1 * torch.arange(1, words + 1, device=trainer.device).float().log()
    trainer.sgd_update(0.0)                    # the gradients are zero: this only renews the kernels' working copies


def prepare(case, seed):
    """A handle with its parameters, and a batch: on the device for the training calls, on the host for the decoders,
    which take host arrays."""
    rows = case["batch"] * (BEAM if case["kind"] == "beam" else 1)
    recipe = dict(_model(case), ids="zipf", batch=case["batch"], len_range=(case["lo"], case["hi"]), seed=seed)
    src, src_len, tgt, tgt_len = I.make_batch(recipe)
    decode = case["kind"] in ("greedy", "beam")
    trainer = binding.Trainer(_model(case), rows, src.shape[1], max(2, case["hi"] if decode else tgt.shape[1]), precision=case["precision"])
    trainer.init_params(seed, SCALE)
    if decode:
        _as_trained(trainer, case, seed)
    batch = (src, src_len) if decode else trainer.upload_batch(src, src_len, tgt, tgt_len)
    return dict(kind=case["kind"], trainer=trainer, batch=batch, max_len=max(2, case["hi"]), steps=0)


def run(state):
    kind, trainer, batch = state["kind"], state["trainer"], state["batch"]
    if kind == "step":
        loss = trainer.train_step(batch)
        return {"loss": loss, "grads": trainer.grads}
    if kind == "async":
        trainer.train_step_async(batch)
        return trainer.grads
    if kind == "update":
        trainer.set_regularization(DROPOUT, SMOOTHING, state["steps"])
        state["steps"] += 1
        trainer.train_step_async(batch)
        trainer.sgd_update(RATE)
        return {"grads": trainer.grads, "params": trainer.params}
    if kind == "eval":
        return trainer.eval_loss(batch)
    if kind == "greedy":
        return trainer.greedy_decode(*batch, state["max_len"])
    return trainer.beam_decode(*batch, state["max_len"], beam=BEAM, length_penalty=LENGTH_PENALTY)


def work(case):
    """Multiply-adds (x2) over the tokens that exist, forward and, for a training step, backward; bytes: every parameter
    in the precision that the matrix cores take, once, and for a training step the fp32 gradients (and the update)."""
    E, H, L, V, B = case["emb"], case["hidden"], case["layers"], case["vocab"], case["batch"]
    tokens = (case["lo"] + case["hi"]) / 2
    Hd = H // 2
    enc = 2 * 2 * 4 * Hd * (E + Hd) + (L - 1) * 2 * 4 * H * 2 * H
    dec = 2 * 4 * H * (E + 2 * H) + (L - 1) * 2 * 4 * H * 2 * H
    attention = 4 * tokens * H + 2 * H * 2 * H
    keys, out = 2 * H * H, 2 * H * V
    params = I.param_count(_model(case))
    operand = 2 if case["precision"] else 4
    if case["kind"] in ("greedy", "beam"):
        rows = B * (BEAM if case["kind"] == "beam" else 1)
        flops = B * tokens * (enc + keys) + rows * case["hi"] * (dec + attention + out)
        weights = params - 2 * V * E
        looked_up = E * (B * tokens + rows * case["hi"])
        return {"bytes": operand * (weights + looked_up) + 4 * B * (tokens + case["hi"]), "flops": flops}
    forward = B * tokens * (enc + keys + dec + attention + out)
    weights = params - 2 * V * E
    read = operand * (weights + 2 * E * B * tokens)
    if case["kind"] == "eval":
        return {"bytes": read, "flops": forward}
    update = 12 * params if case["kind"] == "update" else 0
    return {"bytes": read + 4 * params + update, "flops": 3 * forward}


def tolerance(case):
    """Measured with the sums in another order (other tilings and groupings of the same products) over the listed cases
    and some forty drawn ones.  Gradients: at most 1.2e-3 of their norm and 0.13 of their root mean square with 16-bit
    operands (small batches), 1.7e-7 and 4e-5 in full precision.  Losses 7e-7, normalised search scores 1e-4 with 16-bit
    operands; tokens did not differ."""
    if case["kind"] in ("greedy", "beam"):
        return {"rel": 5e-4 if case["precision"] else 1e-5, "differ": 0.01}
    if case["kind"] == "eval":
        return {"rel": 1e-5}
    return {"rel": 5e-3, "max": 0.5} if case["precision"] else {"rel": 2e-6, "max": 2e-4}
