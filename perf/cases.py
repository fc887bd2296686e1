"""The workloads whose speed matters to a user of this package, as cases that can be timed.

Two kinds of work go through the public plans of ``paper_2411_05288_amd``:

* ``output`` - the sharded output layer (``OutputLayerPlan``): ``step`` is a training step (forward, loss, dH and
  every shard's dW), ``forward`` the loss alone (scoring, evaluation);
* ``embed`` - the sharded input layer (``EmbeddingPlan``): ``step`` is the gather and the scatter-add of its gradient,
  ``forward`` the gather alone.

A case is a dict of plain values.  ``listed()`` holds named ones over the range from the smallest call to the largest
configuration, ``draw()`` gives more of the same ranges.  Inputs are drawn on the GPU from a seed, with the
distributions of the benchmark's configurations (hidden states and gradients N(0, 1), weights N(0, 0.02) or N(0, 0.01),
labels and token ids uniform or Zipf(1.1) over a random permutation of the vocabulary).
"""
import math

import torch

import paper_2411_05288_amd as vp

F32, BF16 = "f32", "bf16"


def _output(name, op, N, h, V, p, dtype, save, labels, algorithm=1, w_std=0.02):
    return {"name": name, "kind": "output", "op": op, "N": N, "h": h, "V": V, "p": p, "dtype": dtype,
            "save_logits": save, "labels": labels, "algorithm": algorithm, "w_std": w_std}


def _embed(name, op, N, h, V, p, dtype, ids):
    return {"name": name, "kind": "embed", "op": op, "N": N, "h": h, "V": V, "p": p, "dtype": dtype, "ids": ids}


def listed():
    return [
        # the smallest training step (the tiny fp32 configuration): launches and latency
        _output("output_tiny_f32", "step", 128, 256, 8192, 2, F32, True, "uniform"),
        # an fp32 step of ordinary size (a model trained or checked in full precision)
        _output("output_f32", "step", 1000, 1024, 32000, 8, F32, True, "uniform"),
        # scoring of a few tokens: the loss alone, bound by reading the weights once
        _output("output_score_few", "forward", 64, 4096, 128256, 8, BF16, False, "zipf"),
        # a small micro-batch of a small model: far fewer rows than the tiles of the large products like
        _output("output_small_batch", "step", 512, 2048, 32000, 4, BF16, True, "uniform"),
        # a vocabulary padded to a multiple of 2p and a token count that is no multiple of anything
        _output("output_ragged", "step", 1999, 3072, 50001, 8, BF16, True, "zipf"),
        # one sequence of 4096 tokens, vocabulary of 32k (the Llama-like configuration)
        _output("output_llama", "step", 4096, 4096, 32000, 8, BF16, True, "uniform"),
        # the same through Algorithm 2 (one barrier)
        _output("output_llama_alg2", "step", 4096, 4096, 32000, 8, BF16, True, "uniform", algorithm=2),
        # vocabulary of 128k, logits kept (the large-vocabulary configuration)
        _output("output_large_vocab", "step", 4096, 4096, 128256, 8, BF16, True, "zipf"),
        # vocabulary of 256k, wide model, logits recomputed in the backward pass (the benchmark's headline)
        _output("output_very_large", "step", 4096, 8192, 256000, 16, BF16, False, "zipf", w_std=0.01),
        # input layer of a small fp32 model
        _embed("embed_small_f32", "step", 512, 1024, 32000, 8, F32, "uniform"),
        # the input-layer configuration: two sequences of 4096 tokens, vocabulary of 256k
        _embed("embed_large_vocab", "step", 8192, 4096, 256000, 8, BF16, "zipf"),
        # a long context (or eight sequences at once) through the input layer
        _embed("embed_long", "step", 32768, 4096, 128256, 8, BF16, "zipf"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A hidden size: a multiple of 64 as a rule, of 8 alone now and then."""
    h = _log_int(rng, lo, hi)
    return max(8, h // 8 * 8) if rng.random() < 0.2 else max(64, h // 64 * 64)


def _rows(case):
    """Rows of a shard: the vocabulary padded to a multiple of 2p and split evenly."""
    m = 2 * case["p"]
    return (case["V"] + m - 1) // m * 2


def draw(rng):
    while True:
        u = rng.random()
        p = rng.choice((1, 2, 4, 8, 16))
        spread = rng.choice(("uniform", "zipf"))
        if u < 0.50:        # bf16 output layer
            alg = 2 if rng.random() < 0.15 else 1
            c = _output("", "forward" if rng.random() < 0.25 else "step", _log_int(rng, 16, 8192), _width(rng, 512, 8192),
                        _log_int(rng, 8000, 256000), p, BF16, rng.random() < 0.6, spread, alg,
                        rng.choice((0.01, 0.02)))
            if c["N"] * c["h"] * c["V"] > 4096 * 8192 * 256000 // 4:
                continue
        elif u < 0.65:      # fp32 output layer
            c = _output("", "forward" if rng.random() < 0.25 else "step", _log_int(rng, 16, 2048), _width(rng, 64, 2048),
                        _log_int(rng, 2000, 64000), p, F32, rng.random() < 0.6, spread)
            if c["N"] * c["h"] * c["V"] > 1000 * 1024 * 64000:
                continue
        else:               # input layer
            c = _embed("", "forward" if rng.random() < 0.25 else "step", _log_int(rng, 16, 65536), _width(rng, 256, 8192),
                       _log_int(rng, 8000, 256000), p, F32 if rng.random() < 0.2 else BF16, spread)
            if p * c["N"] * c["h"] > 1 << 31 or c["N"] * c["h"] >= 1 << 29:
                continue
        if _rows(c) * c["h"] > 1 << 30 or c["N"] * (_rows(c) + 64) >= 1 << 31:
            continue
        if (c["p"] - 1) * _rows(c) >= c["V"]:
            continue
        del c["name"]
        return c


# --------------------------------------------------------------------------- inputs

def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + stream)
    return g


def _normal(shape, std, dtype, seed, stream):
    x = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=_generator(seed, stream))
    return x if dtype == F32 else x.to(torch.bfloat16)


def _ids(n, V, spread, seed, stream):
    g = _generator(seed, stream)
    if spread == "uniform":
        return torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int64)
    cdf = torch.cumsum(torch.arange(1, V + 1, device="cuda", dtype=torch.float64) ** -1.1, 0)
    u = torch.rand((n,), generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
    rank = torch.searchsorted(cdf, u).clamp_(max=V - 1)
    return torch.randperm(V, generator=g, device="cuda", dtype=torch.int64)[rank]


def prepare(case, seed):
    rows, p, N, h, dt = _rows(case), case["p"], case["N"], case["h"], case["dtype"]
    if case["kind"] == "output":
        H = _normal((N, h), 1.0, dt, seed, 1)
        W = [_normal((rows, h), case["w_std"], dt, seed, 100 + r) for r in range(p)]
        labels = _ids(N, case["V"], case["labels"], seed, 2)
        plan = vp.OutputLayerPlan(H, W, labels, case["save_logits"], vocab_size=case["V"], algorithm=case["algorithm"])
    else:
        tables = [_normal((rows, h), 0.02, dt, seed, 100 + r) for r in range(p)]
        grad = _normal((N, h), 1.0, dt, seed, 3)
        plan = vp.EmbeddingPlan(tables, _ids(N, case["V"], case["ids"], seed, 2), grad)
    return {"kind": case["kind"], "op": case["op"], "plan": plan}


def run(state):
    plan = state["plan"]
    if state["kind"] == "output":
        if state["op"] == "step":
            plan.step()
        else:
            plan.forward()
        r = plan.result()
        out = {"loss": r.loss, "loss_rows": r.loss_rows, "global_max": r.global_max, "global_sumexp": r.global_sumexp,
               "local_max": r.local_max, "local_sumexp": r.local_sumexp, "local_target": r.local_target}
        if state["op"] == "step":
            out["dH"], out["dW"] = r.dH, r.dW
        if r.logits is not None:
            out["logits"] = r.logits
        elif plan.algorithm == 2 and state["op"] == "forward":
            out["dH"] = r.dH            # Algorithm 2 has the input gradient when its barrier is over
        return out
    plan.forward()
    if state["op"] == "step":
        plan.backward()
        return {"out": plan.out, "dtable": plan.dtable}
    return {"out": plan.out}


# --------------------------------------------------------------------------- what a pass cannot do without

def work(case):
    N, h, V, p = case["N"], case["h"], case["V"], case["p"]
    e = 4 if case["dtype"] == F32 else 2
    step = case["op"] == "step"
    if case["kind"] == "output":
        # H, W and the labels in; statistics, loss, kept logits and, in a step, dH and dW out
        b = e * (N * h + V * h) + 8 * N + 4 * N * (3 * p + 3)
        # one product in the forward pass, two in the backward pass, a third where the logits are formed again;
        # Algorithm 2 forms softmax' W already in the forward pass
        products = 1 + (1 if case["algorithm"] == 2 else 0)
        if case["save_logits"]:
            b += e * N * V
        if step:
            b += 4 * (N * h + V * h)
            products = 3 if case["save_logits"] else 4
        elif case["algorithm"] == 2:
            b += 4 * N * h
        return {"bytes": b, "flops": 2 * products * N * h * V}
    # the full-size output of every shard, the rows of the table that occur (at most N of them) and the ids; in the
    # backward pass the gradient rows and the rows of the table gradient that change, read and written
    touched = min(N, V) if case["ids"] == "uniform" else min(V, max(1, N // 3))
    b = p * N * h * e + touched * h * e + 8 * N
    flops = 0
    if step:
        b += N * h * e + 2 * touched * h * 4 + 8 * N
        flops = N * h
    return {"bytes": b, "flops": flops}


def tolerance(case):
    if case["kind"] == "embed":
        return "exact"          # a copy, and sums in token order from the value that is there
    # Seen against the same pass in 64 bits on the listed cases: fp32 up to 1.3e-6 (sums of exponentials), largest
    # difference 1.3e-5; bf16 1.7e-3 (kept logits, rounded once) and 5.8e-3 (single elements of dW).
    if case["dtype"] == F32:
        return {"rel": 6e-6, "max": 1e-4}
    return {"rel": 7e-3, "max": 3e-2}
