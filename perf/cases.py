"""The work that users of this library have it do, as timed cases: training steps (oases_forward + oases_backward) and
forward passes of one tensor-model-parallel rank's share of a transformer layer stack.

A case is the keyword set of `binding.make_cfg` (layer family, sizes, partition, sub-batches, dropout rates) plus what the
caller chooses per pass: forward only or a whole training step, one stream or two, stored activations or recomputation,
with or without peer sums at the reduction points.
"""
import math

import torch

from paper_2305_16121_amd import binding as B


def _case(name, **over):
    c = dict(name=name, arch="gpt", hidden=0, n_heads=0, seq=0, batch=0, tp=1, n_sub=1, n_layers=1, causal=1, dropout_p=0.0,
             attn_dropout_p=0.0, ffn_hidden=0, w_sigma=0.02, step="train", streams=2, recompute=False, peers=False)
    c.update(over)
    return c


def listed():
    return [
        # the smallest layer: latency of some forty dependent launches (debugging, unit-sized runs, small ranks)
        _case("gpt_h512", hidden=512, n_heads=8, seq=128, batch=4, tp=2, n_sub=2, causal=0),
        # a two-layer stack at the width of the 340 M-parameter models, short sequences
        _case("gpt_h1024_two_layers", hidden=1024, n_heads=16, seq=512, batch=8, tp=4, n_sub=2, n_layers=2, dropout_p=0.1),
        # a 1.3 B-parameter model's layer
        _case("gpt_h2048", hidden=2048, n_heads=32, seq=1024, batch=8, tp=4, n_sub=2, dropout_p=0.1),
        # the benchmark's layer: 7 B-parameter width on eight ranks
        _case("gpt_h4096", hidden=4096, n_heads=32, seq=2048, batch=4, tp=8, n_sub=2, dropout_p=0.1),
        # the largest: 65 B-parameter width, more sub-batches than sequences (a sub-batch is half a sequence)
        _case("gpt_h8192_chunks", hidden=8192, n_heads=64, seq=2048, batch=2, tp=8, n_sub=4, dropout_p=0.1, w_sigma=0.01),
        # the RMSNorm / rotary / SwiGLU layer at 7 B-parameter width: FFN columns per rank are no multiple of a tile
        _case("llama_h4096", arch="llama", hidden=4096, n_heads=32, seq=2048, batch=4, tp=8, n_sub=2, ffn_hidden=11008),
        # the same family, two layers, activations recomputed inside the backward pass
        _case("llama_h1024_recompute", arch="llama", hidden=1024, n_heads=16, seq=512, batch=4, tp=4, n_sub=2, n_layers=2, dropout_p=0.1,
              ffn_hidden=2816, recompute=True),
        # post-LayerNorm layers, every key visible to every query, dropout on the attention probabilities
        _case("bert_h1024", arch="bert", hidden=1024, n_heads=16, seq=512, batch=4, tp=4, n_sub=2, n_layers=2, causal=0, dropout_p=0.1,
              attn_dropout_p=0.1),
        # memory-saving mode next to other ranks: recomputation, and a peer sum read at all four reduction points
        _case("gpt_h4096_recompute_peers", hidden=4096, n_heads=32, seq=2048, batch=4, tp=8, n_sub=2, dropout_p=0.1, recompute=True, peers=True),
        # odd sizes: 200-token sequences, three sub-batches, three layers
        _case("gpt_h1024_ragged", hidden=1024, n_heads=8, seq=200, batch=3, tp=2, n_sub=3, n_layers=3, dropout_p=0.2),
        # evaluation: forward only, no dropout, one stream
        _case("gpt_h2048_forward", hidden=2048, n_heads=32, seq=1024, batch=8, tp=4, n_sub=2, step="forward", streams=1),
        # few tokens through the widest layer: bound by reading weights and updating gradients
        _case("gpt_h12288_short", hidden=12288, n_heads=96, seq=64, batch=2, tp=8, n_sub=2, dropout_p=0.1, w_sigma=0.01),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        arch = rng.choice(["gpt", "gpt", "llama", "bert"])
        d = rng.choice([64, 128])
        tp = rng.choice([1, 2, 3, 4, 4, 8, 8])
        heads = round(_log_uniform(rng, 1, 12)) * tp
        hidden = d * heads
        if not 256 <= hidden <= 12288:
            continue
        seq = 8 * round(_log_uniform(rng, 8, 256))      # 64 .. 2048 in steps of 8: mostly no multiple of a tile
        batch = rng.randint(1, 8)
        causal = 0 if arch == "bert" else 1
        n_sub = rng.choice([n for n in (1, 2, 2, 3, 4) if batch % n == 0 or (causal and n % batch == 0 and seq % (8 * (n // batch)) == 0)])
        ffn = 32 * tp * max(1, round(8 * hidden / 3 / tp / 32)) if arch == "llama" else 0
        c = _case("drawn", arch=arch, hidden=hidden, n_heads=heads, seq=seq, batch=batch, tp=tp, n_sub=n_sub, n_layers=rng.choice([1, 1, 2, 3]),
                  causal=causal, dropout_p=rng.choice([0.0, 0.1, 0.1, 0.2]), attn_dropout_p=rng.choice([0.0, 0.0, 0.0, 0.1]),
                  ffn_hidden=ffn, w_sigma=round(0.9 / math.sqrt(hidden), 4), step=rng.choice(["train", "train", "train", "forward"]),
                  streams=rng.choice([1, 2, 2]), peers=rng.random() < 0.25)
        c["recompute"] = c["step"] == "train" and rng.random() < 0.2
        del c["name"]
        if work(c)["flops"] <= most and _workspace_estimate(c) <= 8 << 30:
            return c


def _widths(c):
    """hp, fp, fw: attention width, FFN inner width and columns of the first FFN product of this rank."""
    hp = c["hidden"] // c["tp"]
    fp = (c["ffn_hidden"] or 4 * c["hidden"]) // c["tp"]
    return hp, fp, 2 * fp if c["arch"] == "llama" else fp


def _workspace_estimate(c):
    hp, fp, fw = _widths(c)
    return c["n_layers"] * c["batch"] * c["seq"] * (48 * c["hidden"] + 16 * hp + 6 * fw)


def _param_shapes(c):
    h = c["hidden"]
    hp, fp, fw = _widths(c)
    s = {"wqkv": (h, 3 * hp), "wo": (hp, h), "w1": (h, fw), "w2": (fp, h), "ln1_g": (h,), "ln2_g": (h,)}
    if c["arch"] != "llama":
        s.update(bqkv=(3 * hp,), bo=(h,), b1=(fp,), b2=(h,), ln1_b=(h,), ln2_b=(h,))
    return s


class State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, sigma=1.0, mean=0.0, dtype=torch.float32):
        return torch.randn(shape, generator=gen, device="cuda").mul_(sigma).add_(mean).to(dtype)

    s = State()
    s.train = case["step"] == "train"
    flags = (B.FLAG_RECOMPUTE if case["recompute"] else 0) | (B.FLAG_SERIALISE if case["streams"] == 1 else 0)
    s.handle = B.Handle(B.make_cfg(case, rank=case["tp"] - 1, seed=seed, flags=flags))
    shapes = _param_shapes(case)
    s.weights, s.grads, s.grad_buffers = [], [], []
    for _ in range(case["n_layers"]):
        w = {}
        for k, shape in shapes.items():
            if len(shape) == 2:
                w[k] = normal(shape, case["w_sigma"], dtype=torch.bfloat16)
            else:
                w[k] = normal(shape, 0.02, 1.0 if k.endswith("_g") else 0.0)
        s.weights.append(w)
        if s.train:      # one buffer for the gradients of a layer, as data-parallel training keeps them
            sizes = {k: -(-math.prod(v) // 64) * 64 for k, v in shapes.items()}
            flat = torch.zeros(sum(sizes.values()), device="cuda")
            parts = dict(zip(sizes, flat.split(list(sizes.values()))))
            s.grads.append({k: parts[k][:math.prod(v)].view(v) for k, v in shapes.items()})
            s.grad_buffers.append(flat)
    rows = (case["batch"] * case["seq"], case["hidden"])
    s.x, s.y = normal(rows), torch.empty(rows, device="cuda")
    if s.train:
        s.dy, s.dx = normal(rows), torch.empty(rows, device="cuda")
    s.peers = None
    if case["peers"]:
        points = ("fwd_attn", "fwd_ffn", "bwd_ffn", "bwd_attn") if s.train else ("fwd_attn", "fwd_ffn")
        s.peers = [{k: normal(rows, 0.1) for k in points} for _ in range(case["n_layers"])]
    s.workspace = torch.empty(s.handle.workspace_bytes, dtype=torch.uint8, device="cuda")
    s.comm = torch.cuda.Stream() if case["streams"] == 2 else None
    return s


def run(s):
    compute = torch.cuda.current_stream()
    comm = s.comm or compute
    s.handle.forward(s.weights, s.x, s.y, s.workspace, peers=s.peers, s_compute=compute, s_comm=comm)
    out = {"y": s.y}
    if s.train:
        for flat in s.grad_buffers:
            flat.zero_()
        s.handle.backward(s.weights, s.x, s.dy, s.dx, s.grads, s.workspace, peers=s.peers, s_compute=compute, s_comm=comm)
        out.update(dx=s.dx, grads=s.grads)
    return out


def work(case):
    M, h, L = case["batch"] * case["seq"], case["hidden"], case["n_layers"]
    hp, fp, fw = _widths(case)
    train = case["step"] == "train"
    flops = 2.0 * M * h * (4 * hp + fw + fp) + (2.0 if case["causal"] else 4.0) * M * case["seq"] * hp
    weights = grads = 0
    for shape in _param_shapes(case).values():
        n = math.prod(shape)
        weights += n * (2 if len(shape) == 2 else 4)
        grads += n * 4
    points = (4 if train else 2) if case["peers"] else 0
    # x, dy read, y, dx written; the backward pass costs twice the forward's products
    nbytes = L * (weights + (grads if train else 0) + points * M * h * 4) + (4 if train else 2) * M * h * 4
    return {"bytes": nbytes, "flops": flops * L * (3 if train else 1)}


def tolerance(case):
    # bf16 operands, fp32 sums.  Measured: against the definition in 64 bits the largest relative error of an output is
    # 3e-3 to 8e-3 (QKV weight gradients; y 4e-4 to 2e-3); against the same path with its rows split and summed in another
    # order (n_sub = 1) up to 3.8e-3.
    return {"rel": 1.5e-2}
