"""Measured cases: what a program using this package has it do, through the entry points it would call.

Two kinds of case:

  "step"   one LOMO step over a list of independent tensors that the caller owns (LomoStep): every linear tensor with its
           saved input X and output gradient dY, its RMSNorm gains, optionally the embedding table and the output projection.
           Options: how the clipping coefficient is formed ("run": one host read-back; "async": on the device; "clip_value":
           the single pass that clips by value) and the route of the norm pass.
  "train"  one fine-tuning step of a decoder-only model from token ids (LomoTrainer around LomoFineTuneStep): forward,
           loss, backward walk, fused updates, the loss read by the host.  Options: global or grouped norm, activations
           checkpointed or kept, hand-on gradients kept.

Widths are those of the LLaMA shapes the package is configured, tested and benchmarked with (7B, 13B, 65B layers) and two
generic smaller ones; depths are cut to what shows a layer's work and the model's head and tail together.  Token counts run
from one short sequence to eight sequences of 1024, odd counts among them.
"""
from __future__ import annotations

import math

import torch

import paper_2306_09782_amd as L
from paper_2306_09782_amd.chain import LomoFineTuneStep, LomoTrainer
from paper_2306_09782_amd.step import LomoStep

DEVICE = "cuda:0"

# hidden width, heads of width 128, feed-forward width
WIDTHS = {"1k": (1024, 8, 2816), "2k": (2048, 16, 5504), "7b": (4096, 32, 11008), "13b": (5120, 40, 13824),
          "65b": (8192, 64, 22016)}


def _step(name, width, tokens, layers, vocab, mode, norm="direct"):
    return {"name": name, "kind": "step", "width": width, "tokens": tokens, "layers": layers, "vocab": vocab, "mode": mode,
            "norm": norm}


def _train(name, width, batch, seq, layers, vocab, norm, keep_activations=False, keep_handons=False):
    return {"name": name, "kind": "train", "width": width, "batch": batch, "seq": seq, "layers": layers, "vocab": vocab,
            "norm": norm, "keep_activations": keep_activations, "keep_handons": keep_handons}


def listed():
    return [
        # one small adapter-sized tensor: the smallest call, where launches and the host round trip are the time
        _step("one_linear", "1k", 512, 0, 0, "run"),
        # a small model's layer and vocabulary ends on a batch of packed sequences whose token count is odd
        _step("step_2k_odd_tokens", "2k", 777, 1, 32000, "run"),
        # one 7B layer at the batch of the paper's memory profile (8 x 512 tokens), coefficient formed on the device
        _step("step_7b_layer", "7b", 4096, 1, 0, "async"),
        # the same layer when padding has been removed from the batch: an odd number of tokens
        _step("step_7b_layer_odd_tokens", "7b", 2999, 1, 0, "async"),
        # the single-pass alternative (clip by value) over two layers and both vocabulary-sized tensors
        _step("step_7b_clip_value", "7b", 4096, 2, 32000, "clip_value"),
        # a 65B layer at 4 x 512 tokens with the library choosing the route of the norm pass
        _step("step_65b_layer_auto", "65b", 2048, 1, 0, "async", "auto"),
        # a small model on short sequences: many small kernels
        _train("train_1k_2x128", "1k", 2, 128, 4, 32000, "global"),
        # the batch of the paper's throughput table: one sequence of 1024 tokens
        _train("train_7b_1x1024", "7b", 1, 1024, 4, 32000, "global"),
        # a ragged batch (3 x 320) and a vocabulary with eight added tokens
        _train("train_7b_3x320", "7b", 3, 320, 4, 32008, "grouped"),
        # the batch of the paper's memory profile, single backward walk
        _train("train_7b_8x512", "7b", 8, 512, 4, 32000, "grouped"),
        # long context: one sequence of 8192 tokens, where attention matters
        _train("train_7b_1x8192", "7b", 1, 8192, 2, 32000, "grouped"),
        # the largest batch, memory spent to avoid recomputation
        _train("train_13b_8x1024_kept", "13b", 8, 1024, 3, 32000, "global", True, True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same ranges: token counts over their logarithm, odd ones among them."""
    most = max(work(c)["flops"] for c in listed())
    while True:
        if rng.random() < 0.5:
            width = rng.choice(["1k", "2k", "7b", "7b", "13b", "65b"])
            mode = rng.choice(["run", "async", "clip_value"])
            case = _step("", width, _log_int(rng, 200, 8192), rng.choice([1, 1, 2]), rng.choice([0, 32000, 32008]), mode,
                         rng.choice(["direct", "direct", "auto"]) if mode != "clip_value" else "direct")
        else:
            width = rng.choice(["1k", "2k", "7b", "7b", "13b"])
            seq = 64 * _log_int(rng, 2, 64)
            batch = rng.choice([1, 2, 3, 4, 5, 8])
            keep = rng.choice([False, False, True])
            norm = rng.choice(["global", "grouped"])
            case = _train("", width, batch, seq, rng.choice([1, 2, 3]), rng.choice([32000, 32000, 32008]), norm, keep,
                          keep and norm == "global" and rng.random() < 0.5)
            if batch * seq > 8192:
                continue
        del case["name"]
        if work(case)["flops"] <= most:
            return case


# ------------------------------------------------------------------------------------------------------- inputs


class _Source:
    """Seeded values on the GPU."""

    def __init__(self, seed):
        self.gen = torch.Generator(device=DEVICE)
        self.gen.manual_seed(int(seed))

    def normal(self, shape, sigma):
        return torch.randn(shape, generator=self.gen, device=DEVICE, dtype=torch.float16).mul_(sigma)

    def token_ids(self, n, vocab):
        """Token ids as text has them: frequency falling as rank ** -1.1, ranks spread over the vocabulary."""
        p = torch.arange(1, vocab + 1, device=DEVICE, dtype=torch.float32).pow_(-1.1)
        ranks = torch.multinomial(p, n, replacement=True, generator=self.gen)
        return torch.randperm(vocab, generator=self.gen, device=DEVICE)[ranks].to(torch.int32)


def _linear_shapes(case):
    """(out features, in features) of the case's linear tensors, in backward order."""
    H, _, F = WIDTHS[case["width"]]
    if case["layers"] == 0:
        return [(H, H)]
    layer = [(H, F), (F, H), (F, H)] + [(H, H)] * 4
    return ([(case["vocab"], H)] if case["vocab"] else []) + layer * case["layers"]


def _prepare_step(case, seed):
    src = _Source(seed)
    H, _, _ = WIDTHS[case["width"]]
    T, scale = case["tokens"], 65536.0
    f16 = dict(dtype=torch.float16, device=DEVICE)
    tensors, n_params = [], 0
    for N, K in _linear_shapes(case):
        tensors.append({"kind": "linear", "X": src.normal((T, K), 1.0), "dY": src.normal((T, N), 1e-3 * scale),
                        "W": src.normal((N, K), 0.02), "dX": torch.empty(T, K, **f16)})
        n_params += N * K
    for _ in range(2 * case["layers"]):
        tensors.append({"kind": "vector", "X": src.normal((T, H), 1.0), "dY": src.normal((T, H), 1e-3 * scale),
                        "W": torch.ones(H, **f16)})
    if case["vocab"]:
        tensors.append({"kind": "embedding", "ids": src.token_ids(T, case["vocab"]), "dY": src.normal((T, H), 1e-3 * scale),
                        "W": src.normal((case["vocab"], H), 0.02)})
    stepper = LomoStep(DEVICE, max_T=T, max_H=H, norm_algorithm=case["norm"])
    # a learning rate whose clipped update moves the fp16 weights (a few of their last places)
    lr = 1e-4 * math.sqrt(n_params)
    return {"case": case, "stepper": stepper, "tensors": tensors, "lr": lr, "scale": scale}


def _run_step(state):
    stepper, tensors, mode = state["stepper"], state["tensors"], state["case"]["mode"]
    out = {}
    if mode == "run":
        out["norm"] = stepper.run(tensors, state["lr"], state["scale"])["norm"]
    elif mode == "async":
        stepper.run_async(tensors, state["lr"], state["scale"])
        out["clip_and_norm"] = stepper.scalars[:16].view(torch.float64)
    else:
        stepper.clip_value_pass(tensors, 1e-2, 1.0 / state["scale"], 0.05)
        out["flags"] = stepper.flags[:len(tensors) + 1]
    out["W"] = [t["W"] for t in tensors]
    out["dX"] = [t["dX"] for t in tensors if t["kind"] == "linear"]
    return out


def _prepare_train(case, seed):
    src = _Source(seed)
    H, heads, F = WIDTHS[case["width"]]
    n, V, B, s = case["layers"], case["vocab"], case["batch"], case["seq"]
    sigma = 0.02 * math.sqrt(4096.0 / H)
    shapes = [("W_qkv", (3 * H, H)), ("W_o", (H, H)), ("W_gu", (2 * F, H)), ("W_d", (H, F))]
    per_layer = sum(a * b for _, (a, b) in shapes)
    # all weight matrices of the model in one allocation, each parameter a view of it
    flat = torch.empty(n * per_layer + 2 * V * H, dtype=torch.float16, device=DEVICE)
    gains = torch.ones(2 * n + 1, H, dtype=torch.float16, device=DEVICE)
    at = 0

    def take(shape, std):
        nonlocal at
        w = flat[at:at + shape[0] * shape[1]].view(shape)
        at += shape[0] * shape[1]
        return w.normal_(0.0, std, generator=src.gen)

    layers = []
    for i in range(n):
        p = {k: take(shape, sigma) for k, shape in shapes}
        p["w1"], p["w2"] = gains[2 * i], gains[2 * i + 1]
        layers.append(p)
    params = {"W_lm": take((V, H), sigma), "W_emb": take((V, H), 1.0), "w_f": gains[2 * n], "layers": layers}
    ids = src.token_ids(B * s, V)
    targets = torch.roll(ids, -1)
    targets[s - 1::s] = -100                      # no next token behind the last one of a sequence
    angle = (torch.arange(s, device=DEVICE, dtype=torch.float64)[:, None]
             * 10000.0 ** (-torch.arange(64, device=DEVICE, dtype=torch.float64) / 64.0)[None, :])
    step = LomoFineTuneStep(DEVICE, B, s, H, F, heads, n, V, norm=case["norm"], checkpoint=not case["keep_activations"],
                            keep_handons=case["keep_handons"])
    trainer = LomoTrainer(step, lr=3e-2, loss_scale=65536.0, growth_interval=1 << 30)
    return {"case": case, "trainer": trainer, "step": step, "params": params, "flat": flat, "gains": gains, "ids": ids,
            "targets": targets, "cos": torch.cos(angle).float().contiguous(), "sin": torch.sin(angle).float().contiguous()}


def _run_train(state):
    step, n = state["step"], state["case"]["layers"]
    res = state["trainer"].train_step(state["ids"], state["targets"], state["params"], state["cos"], state["sin"])
    norms = res["group_norms"] if state["case"]["norm"] == "grouped" else [res["norm"]]
    return {"loss": res["loss"], "norms": norms, "weights": state["flat"], "gains": state["gains"],
            "logit_gradient": step.logits, "token_loss": step.token_loss, "embedding_gradient": step.chain.grad_in(n)}


def prepare(case, seed):
    return _prepare_step(case, seed) if case["kind"] == "step" else _prepare_train(case, seed)


def run(state):
    return _run_step(state) if state["case"]["kind"] == "step" else _run_train(state)


# ------------------------------------------------------------------------------------------------ work, tolerance


def work(case):
    """Bytes: every input read once, every output written once, in fp16.  Flops: the contractions (and attention's
    products at or below the diagonal) that the chosen options ask for."""
    H, heads, F = WIDTHS[case["width"]]
    if case["kind"] == "step":
        T, shapes = case["tokens"], _linear_shapes(case)
        passes = 2 if case["mode"] == "clip_value" else 3           # (norm), dgrad, update
        flops, nbytes = 0.0, 0.0
        for N, K in shapes:
            direct = 2.0 * T * N * K
            norm = min(direct, 1.0 * T * T * (N + K)) if case["norm"] == "auto" else direct
            flops += 2 * direct + (norm if passes == 3 else 0.0)
            nbytes += 2.0 * (2 * T * K + T * N + 2 * N * K)
        nbytes += 2 * case["layers"] * 2.0 * (2 * T * H + 2 * H)
        if case["vocab"]:
            nbytes += 2.0 * T * H + 4.0 * T + 2 * 2.0 * min(T, case["vocab"]) * H / 3
        return {"bytes": nbytes, "flops": flops}
    n, V, B, s = case["layers"], case["vocab"], case["batch"], case["seq"]
    T = B * s
    layer = H * (3 * H + H + 2 * F + F)
    linear = n * layer + V * H
    walks = 2 if case["norm"] == "global" and not case["keep_handons"] else 1
    again = 0 if case["keep_activations"] else n * (layer - F * H) * walks - (layer - F * H)
    flops = 2.0 * T * (linear + again + 2 * linear + walks * linear)
    pairs = 0.5 * s * (s + 1) * B * heads * 2.0 * 128                # one product over the causal pairs
    forwards = n + (0 if case["keep_activations"] else n * walks - 1)
    flops += pairs * (2 * forwards + 5 * walks * n)
    params = n * layer + V * H
    nbytes = 2.0 * (2 * params + 3 * T * H + 2 * T * V) + 2.0 * n * T * H
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """fp16 storage, fp32 sums.  Four times what the same kernels show with every contraction summed in reverse order:
    "step", one rounding of each output: relative 3e-5, one fp16 last place (1e-3) at most; "train", where gradients pass
    through every layer's fp16 tensors forwards and back: relative 2e-3, 2.4e-2 at most."""
    if case["kind"] == "step":
        return {"rel": 1.2e-4, "max": 4e-3}
    return {"rel": 8e-3, "max": 0.1}
