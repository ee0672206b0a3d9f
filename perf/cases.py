"""The training work this library is used for, as cases that can be timed: one optimizer step of the encoder (masked-LM) or
of the encoder-decoder (translation) model through `Worker` and `PairWorker`, forward, loss, backward, accumulation over the
step's micro-batches, normalisation and Adam, from the smallest models and batches to the largest.

A case is a dict of plain values:
  kind      "encoder" (Worker) or "pairs" (PairWorker)
  model     a key of synth.MODELS / synth.S2S_MODELS
  compute   "bf16" or "fp32"
  micro     sequences (pairs) of every micro-batch of the step, e.g. "8+24+56" (gradients accumulate, one update)
  L, Lt     padded length (source side; Lt: target side of pairs)
  lo        shortest real length as a share of the padded one: a batch's lengths run evenly from lo * L to L, in ascending
            order, as the batcher leaves them (1.0: no padding)
  dropout   dropout rate
  loop      0: the batches are on the GPU and a pass is one train_step; n > 0: a pass is Worker.train over n updates from
            host micro-batches (upload, learning-rate schedule, step, loss read back)
"""
import math

import numpy as np
import torch

from paper_2009_14783_amd import binding as hs
from paper_2009_14783_amd import synth
from paper_2009_14783_amd.step import PairWorker, Worker

# a run that was resumed after 1000 updates, still in the warm-up: learning rates, and the size of the running gradient averages
DONE = 1000
ADAM = {"encoder": dict(lr=1e-5, beta1=0.9, beta2=0.999, eps=1e-8), "pairs": dict(lr=1e-4, beta1=0.9, beta2=0.98, eps=1e-9)}
SCHEDULE = dict(max_lr=1e-4, warmup=10000, total=1000000)
MOMENT = {"encoder": 5e-2, "pairs": 3e-3}


def _enc(model, micro, L, lo=1.0, dropout=0.0, compute="bf16", loop=0):
    return dict(kind="encoder", model=model, compute=compute, micro=micro, L=L, lo=lo, dropout=dropout, loop=loop)


def _pairs(model, micro, L, Lt, lo=0.5, dropout=0.0, compute="bf16"):
    return dict(kind="pairs", model=model, compute=compute, micro=micro, L=L, Lt=Lt, lo=lo, dropout=dropout, loop=0)


def listed():
    return [
        # the reference-precision runs on toy models that a new set-up is checked with: launches and host time only
        dict(_enc("tiny", "4", 64, lo=0.25, compute="fp32"), name="tiny_fp32"),
        dict(_pairs("s2s_tiny", "6", 24, 32, lo=0.3, compute="fp32"), name="s2s_tiny_fp32"),
        # a worker with little memory: two passes over a few short sequences, ragged, then the update
        dict(_enc("bert_base", "3+2", 88, lo=0.6), name="bert_base_small"),
        # pre-training at 128 tokens under a cap of 8192 tokens (the benchmark's step), without and with BERT's dropout
        dict(_enc("bert_base", "64", 128), name="bert_base_128"),
        dict(_enc("bert_base", "64", 128, dropout=0.1), name="bert_base_128_drop"),
        # one batch of a corpus of mixed lengths: the bucket of 385..448 tokens under a cap of 16384 real tokens
        dict(_enc("bert_base", "39", 448, lo=0.86), name="bert_base_varlen"),
        # unequal shares of one global batch, accumulated and normalised by 88
        dict(_enc("bert_base", "8+24+56", 256), name="bert_base_hetero"),
        # the training loop from host data: two updates with upload, schedule and loss report
        dict(_enc("bert_base", "32", 128, lo=0.5, loop=2), name="bert_base_loop"),
        # the largest model: four passes of 32 x 512, one update
        dict(_enc("bert_large", "32+32+32+32", 512), name="bert_large_512"),
        # translation: the per-worker 4096 positions as short sentences with the model's dropout, as long sentences, and a
        # small batch
        dict(_pairs("transformer_base", "128", 32, 32, dropout=0.1), name="pairs_32"),
        dict(_pairs("transformer_base", "24", 168, 176), name="pairs_long"),
        dict(_pairs("transformer_base", "10", 24, 32), name="pairs_small"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more step: the toy models in fp32, BERT-base from a few hundred to 16384 positions per micro-batch, BERT-large up
    to 16384, the translation model up to 8192 positions per side; padded lengths are any multiple of 8."""
    what = rng.choice(["tiny", "s2s_tiny", "bert_base", "bert_base", "bert_base", "bert_base", "bert_large", "transformer_base",
                       "transformer_base", "transformer_base"])
    dropout = rng.choice([0.0, 0.0, 0.1])
    lo = rng.choice([1.0, round(rng.uniform(0.3, 1.0), 3)])
    if what == "tiny":
        return _enc(what, str(_log_int(rng, 1, 32)), 8 * rng.randint(1, 8), lo, dropout, "fp32")
    if what == "s2s_tiny":
        return _pairs(what, str(_log_int(rng, 1, 32)), 8 * rng.randint(1, 8), 8 * rng.randint(1, 8), lo, dropout, "fp32")
    if what == "transformer_base":
        L = 8 * _log_int(rng, 2, 32)
        Lt = min(256, max(8, 8 * int(round(L / 8 * rng.uniform(0.7, 1.4)))))
        return _pairs(what, str(max(1, _log_int(rng, 256, 8192) // max(L, Lt))), L, Lt, lo, dropout)
    L = 8 * _log_int(rng, 4, 64)
    n = rng.choice([1, 1, 2, 3]) if what == "bert_base" else rng.choice([1, 2])
    micro = [max(1, _log_int(rng, 256, 16384) // L) for _ in range(n)]
    loop = rng.choice([0, 0, 0, 1]) if what == "bert_base" else 0
    return _enc(what, "+".join(map(str, micro)), L, lo, dropout, "bf16", loop)


def _lens(n, L, lo):
    first = max(1, int(round(lo * L)))
    return [L - (L - first) * (n - 1 - i) // max(1, n - 1) for i in range(n)]


class _State:
    """What a training program holds between steps: the worker (weights, moments, gradient buffer, arenas) and its data; and
    views of the gradient buffer."""

    def __init__(self, worker, data, adam, loop, layout):
        self.worker, self.data, self.adam, self.loop = worker, data, adam, loop
        self.views = _gradient(worker.G, layout)

    def __del__(self):
        self.worker.close()


def _gradient(G, layout):
    """The gradient buffer but for the token embedding: the layers of each stack as rows, and what lies before and behind
    them.  (The embedding's gradient is seen in the first moment, of which it makes the step.  Most of its rows are those of
    tokens that the batch does not hold, and these are smaller than the rounding of the others by orders of magnitude, so that
    in the gradient by itself one row's rounding would be measured by another's size.)"""
    at = {name: off for name, off, _, _ in layout}
    end = max(off + r * c for _, off, r, c in layout)
    first = [name for name, _, _, _ in layout if name.endswith("0.qkv.w") and name[:-len("0.qkv.w")].isalpha()]
    views = {}
    for i, name in enumerate(first):
        stack = name[:-len("0.qkv.w")]
        n = sum(1 for k in at if k.startswith(stack) and k.endswith(".qkv.w"))
        stop = at[first[i + 1]] if i + 1 < len(first) else at.get("head.t.w", end)
        views[stack] = G[at[name]:stop].view(n, -1)
    if "head.t.w" in at:
        views["head"] = G[at["head.t.w"]:]
        views["positions"] = G[at["emb.pos"]:at[first[0]]]
    return views


def prepare(case, seed):
    pairs = case["kind"] == "pairs"
    model = (synth.S2S_MODELS if pairs else synth.MODELS)[case["model"]]
    layout = hs.hs_s2s_param_layout(hs.make_s2s_cfg(**model)) if pairs else hs.hs_param_layout(hs.make_cfg(**model))
    n_params = max(off + r * c for _, off, r, c in layout)
    worker = (PairWorker if pairs else Worker)(model, case["compute"], np.zeros(n_params, dtype=np.float32))
    # weights as synth.init_params makes them but drawn on the GPU: N(0, 0.02), LayerNorm gains around 1; moments of a run in progress
    gen = torch.Generator(device="cuda").manual_seed(seed)
    worker.w.normal_(0.0, 0.02, generator=gen)
    worker.m.normal_(0.0, MOMENT[case["kind"]], generator=gen)
    worker.v.uniform_(4.0 * MOMENT[case["kind"]] ** 2, 16.0 * MOMENT[case["kind"]] ** 2, generator=gen)
    worker.t = DONE
    for name, off, r, c in layout:
        if name.endswith(".g"):
            worker.w[off:off + r * c] += 1.0
    if worker.w_lowp is not None:
        hs.hs_cast_params(worker.w, worker.w_lowp, worker.P, hs.HS_BF16)
    rng = synth.rng_for(seed)
    dist = "uniform" if case["compute"] == "fp32" else "zipf"
    micro, L = [int(b) for b in case["micro"].split("+")], case["L"]
    steps = []
    for t in range(max(1, case["loop"])):
        batches = []
        for i, n in enumerate(micro):
            if pairs:
                # targets of a batch have other lengths than their sources: the same spread, dealt out in another order
                tl = _lens(n, case["Lt"], case["lo"])
                mb = synth.make_pair_batch(rng, _lens(n, L, case["lo"]), tl[n // 2:] + tl[:n // 2], L, case["Lt"], model["vocab"], dist)
            else:
                mb = synth.make_micro_batch(rng, _lens(n, L, case["lo"]), L, model["vocab"], dist)
            if case["dropout"] > 0:
                mb["drop"] = dict(p=case["dropout"], seed=seed, stream=64 * t + i)
            batches.append(mb)
        steps.append(batches)
    return _State(worker, steps if case["loop"] else [worker.upload(mb) for mb in steps[0]], ADAM[case["kind"]], case["loop"], layout)


def run(state):
    """One optimizer step (or state.loop updates of the training loop): the updated weights and moments, the gradient that
    was applied (see _gradient) and the loss sums."""
    worker = state.worker
    out = {}
    if state.loop:
        done = worker.t
        out["losses"] = np.asarray(worker.train(state.loop, lambda t: state.data[t - 1 - done], state.adam, SCHEDULE), dtype=np.float32)
    else:
        worker.train_step(state.data, state.adam)
        out["loss_sums"] = worker.loss_buf
    out.update(w=worker.w, m=worker.m, v=worker.v, G=state.views)
    if worker.w_lowp is not None:
        out["w_lowp"] = worker.w_lowp
    return out


def work(case):
    """Forward and backward (twice the forward) of the real tokens, with the masked-LM or the output projection over the
    target positions; weights, moments, gradient and the bf16 copy once per update."""
    micro = [int(b) for b in case["micro"].split("+")]
    updates = max(1, case["loop"])
    flops = 0.0
    if case["kind"] == "pairs":
        m = synth.S2S_MODELS[case["model"]]
        H, F, V = m["hidden"], m["ffn"], m["vocab"]
        n_params = hs.hs_s2s_param_count(hs.make_s2s_cfg(**m))
        for n in micro:
            ls, lt = _lens(n, case["L"], case["lo"]), _lens(n, case["Lt"], case["lo"])
            lt = lt[n // 2:] + lt[:n // 2]
            s, t = sum(ls), sum(lt)
            flops += m["n_enc"] * (s * (8.0 * H * H + 4.0 * H * F) + 4.0 * H * sum(a * a for a in ls))
            flops += m["n_dec"] * (t * (12.0 * H * H + 4.0 * H * F) + s * 4.0 * H * H + 2.0 * H * sum(b * b for b in lt) +
                                   4.0 * H * sum(a * b for a, b in zip(ls, lt)))
            flops += t * 2.0 * H * V
    else:
        m = synth.MODELS[case["model"]]
        H, F, V = m["hidden"], m["ffn"], m["vocab"]
        n_params = hs.hs_param_count(hs.make_cfg(**m))
        for n in micro:
            ls = _lens(n, case["L"], case["lo"])
            flops += m["n_layers"] * (sum(ls) * (8.0 * H * H + 4.0 * H * F) + 4.0 * H * sum(a * a for a in ls))
            flops += sum(synth.n_targets(a) for a in ls) * (2.0 * H * H + 2.0 * H * V)
    # w, m, v read and written, G written; the low-precision copy read and written
    bytes_ = n_params * (28.0 + (4.0 if case["compute"] == "bf16" else 0.0))
    return {"bytes": updates * bytes_, "flops": updates * 3.0 * flops}


def tolerance(case):
    """bf16: activations and their gradients are rounded at every layer (2^-9 each), which comes to 1e-2 of a layer's gradient;
    a single entry is off by that share of its row's or column's size, which can be tens of times the layer's.  fp32: sums
    of 32-bit products in another order, 1e-4.  In the translation model a ReLU gate whose input is within rounding of zero
    falls on one side or the other and moves a unit's gradient as a whole, 2e-3 of the toy model's for one gate."""
    if case["compute"] == "bf16":
        return {"rel": 2.5e-2 if case["kind"] == "pairs" else 2e-2, "max": 0.95}
    return {"rel": 3e-3, "max": 0.5} if case["kind"] == "pairs" else {"rel": 1e-4, "max": 1e-2}
