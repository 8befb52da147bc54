"""Workloads whose speed matters to a user of the training-step library, through its public entry points.

A training case is an interval of a run in its steady state: `steps` mini-batches go through `Model.step`, the loss is
read once at the end (logging), and the weights are handed over on the device (what an evaluation model or a checkpoint
is fed from).  An evaluation case runs consecutive segments through `Model.eval_step` and reads each loss.  Inputs are
synthetic: Zipf-distributed token ids, as frequent ids dominate in text, and weights drawn the way the models are
initialised.
"""
import ctypes

import torch

import paper_1909_06695_amd as P

_FIELDS = ("n_layer", "d_model", "n_head", "d_head", "d_ff", "vocab", "seq_len", "mem_len", "batch", "n_module",
           "rel_pos", "dtype", "optimizer", "schedule", "dropout")


def _case(name=None, *, steps, zipf=1.1, lr=2.5e-4, evaluate=False, **cfg):
    c = dict(mem_len=0, rel_pos=0, dtype=1, optimizer=1, schedule=0, dropout=0.0)
    c.update(cfg)
    c.update(steps=steps, zipf=zipf, lr=lr, evaluate=evaluate)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest model anyone steps: unit-size fp32 with SGD, where a pass is launches and little else.
        _case("tiny-fp32-sgd", n_layer=2, d_model=64, n_head=2, d_head=32, d_ff=256, vocab=256, seq_len=32, batch=4,
              n_module=2, dtype=0, optimizer=0, lr=0.1, steps=3),
        # A small experiment in bf16, with a vocabulary and a segment off every tile size.
        _case("small-odd-vocab", n_layer=3, d_model=128, n_head=2, d_head=64, d_ff=256, vocab=1001, seq_len=96, batch=3,
              n_module=3, steps=4),
        # Training in full fp32 (the parity mode) at an ordinary width.
        _case("decoder-512-fp32", n_layer=6, d_model=512, n_head=8, d_head=64, d_ff=2048, vocab=8192, seq_len=256, batch=4,
              n_module=3, dtype=0, steps=2),
        # One long ragged batch: three streams of 777 tokens, 768 wide, K = 5 over 8 layers.
        _case("decoder-768-ragged", n_layer=8, d_model=768, n_head=12, d_head=64, d_ff=3072, vocab=30011, seq_len=777, batch=3,
              n_module=5, steps=4),
        # The 12-layer character / word decoder, the ordinary size.
        _case("decoder-512", n_layer=12, d_model=512, n_head=8, d_head=64, d_ff=2048, vocab=32768, seq_len=512, batch=16,
              n_module=4, steps=4),
        # The same under the memory-saving schedule (stored inputs, recomputation) with repeatable dropout.
        _case("decoder-512-recompute", n_layer=12, d_model=512, n_head=8, d_head=64, d_ff=2048, vocab=32768, seq_len=512, batch=16,
              n_module=4, schedule=1, dropout=0.125, steps=4),
        # The 16-layer relative-position model of the word-level benchmark: widths off the tile grid, segment memory.
        _case("xl-410", n_layer=16, d_model=410, n_head=10, d_head=41, d_ff=2100, vocab=32768, seq_len=150, mem_len=150, batch=32,
              n_module=4, rel_pos=1, steps=8),
        # The largest plain decoder that the benchmark runs.
        _case("decoder-1024", n_layer=24, d_model=1024, n_head=16, d_head=64, d_ff=4096, vocab=50257, seq_len=1024, batch=8,
              n_module=8, steps=2),
        # The largest relative-position model.
        _case("xl-1024", n_layer=18, d_model=1024, n_head=16, d_head=64, d_ff=4096, vocab=65536, seq_len=384, mem_len=384, batch=16,
              n_module=4, rel_pos=1, zipf=1.05, steps=2),
        # Evaluation of that model on two streams with a memory three times the training length.
        _case("xl-1024-eval", n_layer=18, d_model=1024, n_head=16, d_head=64, d_ff=4096, vocab=65536, seq_len=384, mem_len=1152, batch=2,
              n_module=4, rel_pos=1, zipf=1.05, steps=4, evaluate=True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    """One more training interval or evaluation over the range between the smallest and the largest listed ones."""
    while True:
        kind = rng.choice(("plain", "plain", "relative", "relative", "recompute", "fp32", "evaluate"))
        fp32 = kind == "fp32"
        d_head = rng.choice((64, 64, 64, 32, 41))
        n_head = _log_int(rng, 1, 8 if fp32 else 16)
        if d_head % 2 and n_head % 2:
            n_head += 1
        d = d_head * n_head
        d_ff = rng.choice((2 * d, 4 * d, 4 * d, _log_int(rng, d, 4 * d)))
        n_layer = rng.randint(2, 8 if fp32 else 24)
        seq_len = _log_int(rng, 32, 512 if fp32 else 1024)
        batch = _log_int(rng, 1, max(1, min(64, (2048 if fp32 else 8192) // seq_len)))
        relative = kind == "relative" or (kind in ("recompute", "evaluate") and rng.random() < 0.5)
        c = _case(n_layer=n_layer, d_model=d, n_head=n_head, d_head=d_head, d_ff=d_ff,
                  vocab=_log_int(rng, 256, 16384 if fp32 else 65536), seq_len=seq_len, batch=batch,
                  n_module=rng.randint(1, min(8, n_layer)), rel_pos=int(relative),
                  mem_len=rng.choice((seq_len, seq_len, 2 * seq_len, seq_len // 2)) if relative else 0,
                  dtype=0 if fp32 else 1, optimizer=rng.choice((1, 1, 1, 0)),
                  schedule=int(kind == "recompute"), dropout=0.125 if kind == "recompute" and rng.random() < 0.5 else 0.0,
                  steps=rng.choice((2, 3, 4)), evaluate=kind == "evaluate")
        if c["optimizer"] == 0:
            c["lr"] = 0.05
        w = work(c)
        if w["flops"] <= (1e12 if fp32 else 3.5e13) and w["bytes"] <= 3e10:
            return c


def _param_groups(c):
    """Per parameter group the (count, kind) runs of its blob: w N(0, 0.02^2), g LayerNorm gain, b bias."""
    d, f = c["d_model"], c["d_ff"]
    layer = [(d * 3 * d + d * d + (d * d + 2 * d if c["rel_pos"] else 0), "w"), (d, "g"), (d, "b"), (d * f, "w"), (f, "b"),
             (f * d, "w"), (d, "b"), (d, "g"), (d, "b")]
    K, L = c["n_module"], c["n_layer"]
    return [[(c["vocab"] * d, "w")]] + [layer * n for n in _split(L, K)]


def _split(n_layer, n_module):
    base, rem = divmod(n_layer, n_module)
    sizes = [base] * n_module
    order = list(range(1, n_module - 1)) + [0, n_module - 1]
    for i in range(rem):
        sizes[order[i % n_module]] += 1
    return sizes


def prepare(case, seed):
    """A model with its weights set, mid-training (every gradient ring and segment memory filled), and resident batches."""
    c = case
    gen = torch.Generator(device="cuda").manual_seed(seed)
    model = P.create_model(device="cuda:0", seed=seed, **{k: c[k] for k in _FIELDS})
    weights = []
    for g, runs in enumerate(_param_groups(c)):
        blob = torch.empty(sum(n for n, _ in runs), dtype=torch.float32, device="cuda")
        blob.normal_(0.0, 0.02, generator=gen)
        at = 0
        for n, kind in runs:
            if kind != "w":
                blob[at:at + n] = 1.0 if kind == "g" else 0.0
            at += n
        if blob.numel() != model.param_count(g):
            raise ValueError("parameter group %d has %d elements" % (g, model.param_count(g)))
        _device_params(model, "ouro_set_params", g, blob)
        weights.append(blob)
    torch.cuda.synchronize()
    # resident token batches: contiguous segments where a memory carries over, fresh blocks otherwise
    n, B, T = 4 * c["steps"], c["batch"], c["seq_len"]
    p = torch.arange(1, c["vocab"] + 1, device="cuda", dtype=torch.float64).pow_(-c["zipf"])
    cdf = torch.cumsum(p, 0)
    cdf /= cdf[-1].clone()

    def tokens(*shape):
        u = torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)
        return torch.searchsorted(cdf, u).clamp_(max=c["vocab"] - 1).to(torch.int32)

    if c["mem_len"]:
        stream = tokens(B, n * T + 1)
        tok = stream[:, :-1].reshape(B, n, T).transpose(0, 1).contiguous()
        tgt = stream[:, 1:].reshape(B, n, T).transpose(0, 1).contiguous()
    else:
        block = tokens(n, B, T + 1)
        tok, tgt = block[:, :, :-1].contiguous(), block[:, :, 1:].contiguous()
    s = {"model": model, "case": c, "weights": weights, "batches": list(zip(tok.unbind(0), tgt.unbind(0))), "at": 0}
    warm = -(-c["mem_len"] // T) if c["evaluate"] else max(c["n_module"] + 1, -(-c["mem_len"] // T))
    for _ in range(warm):
        _one(s, False)
    torch.cuda.synchronize()
    return s


def _device_params(model, call, group, blob):
    rc = getattr(model.L, call)(model.h, group, ctypes.c_void_p(blob.data_ptr()), blob.numel(), 1)
    if rc:
        raise P.OuroError(rc, model.L.ouro_last_error().decode())


def _one(s, want_loss):
    tok, tgt = s["batches"][s["at"] % len(s["batches"])]
    s["at"] += 1
    if s["case"]["evaluate"]:
        return s["model"].eval_step(tok, tgt, want_loss=want_loss)
    return s["model"].step(tok, tgt, s["case"]["lr"], want_loss=want_loss)


def run(state):
    s = state
    steps = s["case"]["steps"]
    if s["case"]["evaluate"]:
        return {"losses": [_one(s, True) for _ in range(steps)]}
    loss = None
    for i in range(steps):
        loss = _one(s, i == steps - 1)
    for g, blob in enumerate(s["weights"]):
        _device_params(s["model"], "ouro_get_params", g, blob)
    return {"loss": loss, "weights": s["weights"]}


def work(case):
    """Multiply-adds count 2; causal attention counts visible (query, key) pairs; the backward pass costs twice the forward
    pass, except that memory rows get no input gradient; recomputation, padding and masked pairs count nothing.  Bytes:
    the optimizer's reads and writes of the weights, moments and gradients, the weights handed over, token ids."""
    c = case
    d, f, L, V, T, M, B = (c[k] for k in ("d_model", "d_ff", "n_layer", "vocab", "seq_len", "mem_len", "batch"))
    params = V * d + L * (4 * d * d + 2 * d * f + (d * d if c["rel_pos"] else 0))
    if c["rel_pos"]:
        layer = 2 * d * d + 2 * d * d * (T + M) / T + 2 * d * f
        attn = 6 * d * (M + (T + 1) / 2)
    else:
        layer = 4 * d * d + 2 * d * f
        attn = 4 * d * (T + 1) / 2
    forward = B * T * (2 * (L * layer + V * d) + L * attn)
    element = 4 if c["dtype"] == 0 else 2
    if c["evaluate"]:
        return {"flops": c["steps"] * forward, "bytes": c["steps"] * (params * element + 2 * L * B * M * d * element + 8 * B * T)}
    step = 3 * forward
    if c["rel_pos"]:
        step -= B * T * L * 4 * d * d * M / T
    per_param = 8 + 8 + (16 if c["optimizer"] else 0)      # gradient written and read, weight read and written, two moments
    return {"flops": c["steps"] * step, "bytes": params * (c["steps"] * per_param + 8) + c["steps"] * 8 * B * T}


def tolerance(case):
    """About four times what correct runs differ by.  bf16 intervals against the same intervals in fp32: weights 3e-4 to 9e-4
    in the norm and 0.06 for single elements (an Adam step whose gradient is below the rounding noise goes either way),
    with relative positions 3e-3 and 0.1; evaluation losses 2e-5.  fp32 intervals against the same in another order of
    summation: 6e-7 in the norm; single elements under Adam as in bf16, only fewer."""
    if case["evaluate"]:
        return {"rel": 1e-4 if case["dtype"] else 1e-6}
    if case["dtype"] == 0:
        return {"rel": 5e-6, "max": 0.1 if case["optimizer"] else 1e-3}
    return {"rel": 1.2e-2, "max": 0.4} if case["rel_pos"] else {"rel": 4e-3, "max": 0.25}
