"""What the performance of the virtual-node training step is measured on.

A pass is one training step through the package's own class (`VirtualNodeStep`): partition, every
node's forward and backward pass, the weighted fold of the node gradients, one optimizer update.
A case names a model, the nodes its batch is split into, and how the step is launched:

  launch "units"    what bench.py uses: fused fold, units of up to 32 nodes, a fold window, two streams
         "nodes"    fused fold, node after node (units of one node, window 1), one stream replayed as a graph
         "default"  the constructor without options: node after node, staging vector + accumulate kernel,
                    the default stream, launches made one by one
  input  "device"   the batch lies in device memory
         "host"     the batch lies in pinned host memory and goes through prefetch / step_prefetched

Models are built from the sizes of the repository's configurations and their relatives; node sizes
are written "8x128" (eight nodes of 128) or "48+16+40" (unequal ones, in batch order).
"""
import math
from types import SimpleNamespace

import torch

import paper_2009_09523_amd as vf

# ---------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------


def _mlp(name, dims, batchnorm, dtype, nodes, launch, lr=0.01, input="device"):
    return {"name": name, "kind": "mlp", "dims": dims, "batchnorm": batchnorm, "dtype": dtype, "nodes": nodes,
            "optimizer": "sgdm", "lr": lr, "launch": launch, "input": input}


def _encoder(name, layers, d, heads, ffn, seq, vocab, dtype, nodes, launch):
    return {"name": name, "kind": "encoder", "layers": layers, "d_model": d, "heads": heads, "ffn": ffn, "seq": seq,
            "vocab": vocab, "dtype": dtype, "nodes": nodes, "optimizer": "adam", "lr": 1e-4, "launch": launch,
            "input": "device"}


def _conv(name, img, in_ch, width, blocks, classes, nodes, launch):
    return {"name": name, "kind": "conv", "img": img, "in_ch": in_ch, "width": width, "blocks": blocks,
            "classes": classes, "dtype": "bf16", "nodes": nodes, "optimizer": "sgdm", "lr": 0.01, "launch": launch,
            "input": "device"}


def listed():
    return [
        # the smallest job anybody runs (a digits classifier in fp32): every launch counts
        _mlp("mlp_f32_digits", "784-256-10", False, "f32", "4x16", "units", lr=0.1),
        # fp32 at an ordinary size, widths and node sizes off the powers of two, no options given
        _mlp("mlp_f32_ragged", "784-1000-500-10", True, "f32", "100+56+101", "default", lr=0.1),
        # a classifier on image features as the benchmark launches it, weights resident in cache
        _mlp("mlp_units", "1024-4096-4096-4096-1000", True, "bf16", "8x128", "units"),
        # the same model on a device that got the small share of a heterogeneous job: few rows, unequal nodes
        _mlp("mlp_unequal", "1024-4096-4096-4096-1000", True, "bf16", "48+48+32+32+16+16+48+16", "units"),
        # the literal method: node after node, constant memory
        _mlp("mlp_node_by_node", "1024-4096-4096-4096-1000", True, "bf16", "8x128", "nodes"),
        # few large nodes of odd sizes, batches streamed from host memory
        _mlp("mlp_big_nodes_host", "1024-4096-4096-1000", True, "bf16", "512+301+211", "units", input="host"),
        # the headline configuration: 361 M parameters, global batch 8192 in nodes of 128
        _mlp("mlp_large", "2048-8192-8192-8192-8192-8192-8192-1000", True, "bf16", "64x128", "units"),
        # pre-training of a BERT-like encoder, sequence length 128
        _encoder("encoder_pretrain", 4, 768, 12, 3072, 128, 30522, "bf16", "16x16", "units"),
        # a smaller encoder, sequences cut at 100 tokens, nodes of odd sizes
        _encoder("encoder_ragged", 2, 512, 8, 2048, 100, 9001, "bf16", "16+17+7", "units"),
        # a small encoder in fp32, no options given
        _encoder("encoder_f32", 2, 256, 4, 1024, 64, 4099, "f32", "4+2+3", "default"),
        # a residual network on 32 x 32 colour images
        _conv("conv_units", 32, 3, 64, 2, 10, "8x128", "units"),
        # the same family on 28 x 28 grey images, a narrower network, odd nodes, node after node
        _conv("conv_ragged", 28, 1, 40, 2, 10, "48+33+47", "nodes"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, step):
    """A layer width: mostly a multiple of `step`, one in five any number."""
    w = _log_int(rng, lo, hi)
    return w if rng.random() < 0.2 else max(lo, w // step * step)


def _nodes(rng, batch, most, count):
    """Up to `count` nodes of at most `most` samples, about `batch` of them: equal, or of sizes of their own."""
    n = max(1, min(count, _log_int(rng, 1, count)))
    if rng.random() < 0.5:
        b = max(1, min(most, batch // n))
        return "%dx%d" % (n, b // 8 * 8 if b >= 16 and rng.random() < 0.7 else b)
    n = min(n, 12)
    sizes = [max(1, min(most, int(batch / n * rng.uniform(0.4, 1.6)))) for _ in range(n)]
    return "+".join(str(b // 8 * 8 if b >= 16 and rng.random() < 0.5 else b) for b in sizes)


def draw(rng):
    kind = rng.choices(["mlp", "mlp_f32", "encoder", "encoder_f32", "conv"], [9, 3, 4, 1, 3])[0]
    launch = rng.choices(["units", "nodes", "default"], [6, 2, 2])[0]
    if kind == "mlp":
        literal = launch != "units"
        hidden = rng.randint(1, 3 if literal else 6)
        width = _width(rng, 256, 4096 if literal else 8192, 128)
        dims = [_log_int(rng, 32, 256) * 8]
        dims += [width if rng.random() < 0.7 else _width(rng, 256, width + 1, 8) for _ in range(hidden)]
        dims += [_log_int(rng, 10, 1000)]
        big = rng.random() < 0.25
        nodes = _nodes(rng, _log_int(rng, 64, 1024 if literal else 8192), 1024 if big else 128, 8 if big else 64)
        c = _mlp("", "-".join(map(str, dims)), rng.random() < 0.75, "bf16", nodes, launch,
                 input=rng.choices(["device", "host"], [3, 1])[0])
    elif kind == "mlp_f32":
        dims = [_log_int(rng, 64, 1024)] + [_width(rng, 64, 1024, 8) for _ in range(rng.randint(1, 3))]
        dims += [_log_int(rng, 10, 1000)]
        c = _mlp("", "-".join(map(str, dims)), rng.random() < 0.5, "f32", _nodes(rng, _log_int(rng, 32, 512), 256, 16),
                 launch, lr=0.1)
    elif kind.startswith("encoder"):
        f32 = kind == "encoder_f32"
        heads = rng.randint(2, 6 if f32 else 12)
        usual = rng.random() < 0.6
        seq = rng.choice([32, 64, 128]) if usual else _log_int(rng, 16, 200)
        tokens = _log_int(rng, 256, 2048 if f32 else (32768 if usual and launch == "units" else 8192))
        c = _encoder("", rng.randint(1, 2 if f32 else 4), 64 * heads, heads, 8 * _log_int(rng, 16 * heads, 32 * heads), seq,
                     _log_int(rng, 1000, 30522), "f32" if f32 else "bf16", _nodes(rng, max(1, tokens // seq), 32, 16),
                     launch)
    else:
        img, width, blocks = _log_int(rng, 8, 32), 8 * _log_int(rng, 2, 16), rng.randint(1, 3)
        room = 1024 * 32 * 32 * 64 * 64 * 2 // (img * img * width * width * blocks)     # at most conv_units' work
        c = _conv("", img, rng.choice([1, 3]), width, blocks, rng.choice([10, 100]),
                  _nodes(rng, _log_int(rng, 8, max(9, min(1024, room // 2))), 128, 8), launch)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------
# models, inputs, passes
# ---------------------------------------------------------------------------------------------


def _node_sizes(case):
    if "x" in case["nodes"]:
        n, b = case["nodes"].split("x")
        return [int(b)] * int(n)
    return [int(b) for b in case["nodes"].split("+")]


def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _masked(case):
    return max(1, int(0.15 * case["seq"]))


def _layout(case):
    """(entries, standard deviation or constant) of the flat parameter vector, in order: matrices He-normal,
    embedding tables N(0, 0.02^2), biases 0, normalisation scales 1 and shifts 0."""
    out = []

    def matrix(k, n):
        out.append((k * n, math.sqrt(2.0 / k), 0.0))

    def vectors(n, *values):
        out.extend((n, 0.0, v) for v in values)

    if case["kind"] == "mlp":
        dims = _dims(case)
        for l in range(len(dims) - 1):
            matrix(dims[l], dims[l + 1])
            vectors(dims[l + 1], *((1.0, 0.0) if case["batchnorm"] and l < len(dims) - 2 else (0.0,)))
    elif case["kind"] == "encoder":
        d, f = case["d_model"], case["ffn"]
        out.append(((case["vocab"] + case["seq"]) * d, 0.02, 0.0))
        for _ in range(case["layers"]):
            vectors(d, 1.0, 0.0)
            matrix(d, 3 * d), vectors(3 * d, 0.0)
            matrix(d, d), vectors(d, 0.0)
            vectors(d, 1.0, 0.0)
            matrix(d, f), vectors(f, 0.0)
            matrix(f, d), vectors(d, 0.0)
        vectors(d, 1.0, 0.0)
        matrix(d, case["vocab"]), vectors(case["vocab"], 0.0)
    else:
        c = case["width"]
        for k in [case["in_ch"]] + [c] * (2 * case["blocks"]):
            out.append((9 * k * c, math.sqrt(2.0 / (9 * k)), 0.0))
            vectors(c, 1.0, 0.0)
        matrix(c, case["classes"]), vectors(case["classes"], 0.0)
    return out


def _params(case, gen):
    layout = _layout(case)
    theta = torch.empty(sum(n for n, _, _ in layout), dtype=torch.float32, device="cuda")
    at = 0
    for n, std, value in layout:
        part = theta[at:at + n]
        part.normal_(0.0, std, generator=gen) if std else part.fill_(value)
        at += n
    return theta


def _batch(case, B, gen):
    if case["kind"] != "encoder":
        shape = (B, _dims(case)[0]) if case["kind"] == "mlp" else (B, case["img"], case["img"], case["in_ch"])
        classes = _dims(case)[-1] if case["kind"] == "mlp" else case["classes"]
        x = torch.randn(shape, generator=gen, device="cuda")
        y = torch.randint(classes, (B,), generator=gen, device="cuda", dtype=torch.int32)
        return (x.to(torch.bfloat16) if case["dtype"] == "bf16" else x), y
    # words as in text: the k-th most frequent one with a probability of about 1/k; id 0 stands for a masked word
    T, m = case["seq"], _masked(case)
    u = torch.rand((B, T), generator=gen, device="cuda")
    ids = (case["vocab"] ** u).to(torch.int32).clamp_(1, case["vocab"] - 1)
    where = torch.rand((B, T), generator=gen, device="cuda").argsort(1)[:, :m].sort(1).values
    target = ids.gather(1, where)
    ids.scatter_(1, where, 0)
    return ids, torch.stack([where.to(torch.int32), target], 1).contiguous()


_stream = None


def _the_stream():
    """The one stream of the program (the library puts a second one of its own beside it)."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def _options(case):
    """The constructor's options of a way of launching."""
    if case["launch"] == "units":
        return {"flags": vf.VF_FLAG_FUSED_ACCUMULATE | vf.VF_FLAG_NO_GRAPH | vf.VF_FLAG_OVERLAP, "fold_window": 8,
                "node_group": 32, "stream": _the_stream()}
    if case["launch"] == "nodes":
        return {"flags": vf.VF_FLAG_FUSED_ACCUMULATE, "stream": _the_stream()}
    return {}


def prepare(case, seed):
    """The step object of a training job, its parameters and one batch."""
    nodes = _node_sizes(case)
    B = sum(nodes)
    job = SimpleNamespace(kind=case["kind"], dtype=case["dtype"], optimizer=case["optimizer"], lr=case["lr"],
                          momentum=0.9, beta1=0.9, beta2=0.999, adam_eps=1e-8, bn_eps=1e-5, bn_momentum=0.1, ln_eps=1e-5,
                          node_sizes=tuple(nodes), batch=B, batchnorm=bool(case.get("batchnorm", False)))
    if case["kind"] == "mlp":
        job.dims = tuple(_dims(case))
    elif case["kind"] == "encoder":
        job.n_layers, job.d_model, job.n_heads, job.d_ffn = case["layers"], case["d_model"], case["heads"], case["ffn"]
        job.seq_len, job.vocab, job.n_masked = case["seq"], case["vocab"], _masked(case)
    else:
        job.img, job.in_ch, job.width, job.n_blocks, job.classes = (case["img"], case["in_ch"], case["width"],
                                                                    case["blocks"], case["classes"])
    step = vf.VirtualNodeStep.for_workload(job, **_options(case))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    params = _params(case, gen)
    x, y = _batch(case, B, gen)
    if case["input"] == "host":
        x, y = (t.cpu().pin_memory() for t in (x, y))
    torch.cuda.synchronize()
    return SimpleNamespace(step=step, params=params, x=x, y=y, nodes=nodes, host=case["input"] == "host")


def run(state):
    """One training step: the updated parameters."""
    if state.host:
        state.step.prefetch(state.x, state.y)
        state.step.step_prefetched(state.params, state.nodes)
    else:
        state.step.step(state.params, state.x, state.y, state.nodes)
    return state.params


def work(case):
    """Parameters and optimizer state in and out, the combined gradient out, the batch in; the products of the
    forward pass, of the input gradients (not of the first layer's) and of the weight gradients."""
    B = sum(_node_sizes(case))
    P = sum(n for n, _, _ in _layout(case))
    nbytes = P * 4 * (5 if case["optimizer"] == "sgdm" else 7)
    if case["kind"] == "mlp":
        dims = _dims(case)
        macs = [a * b for a, b in zip(dims, dims[1:])]
        flops = 2 * B * (3 * sum(macs) - macs[0])
        nbytes += B * (dims[0] * (2 if case["dtype"] == "bf16" else 4) + 4)
    elif case["kind"] == "encoder":
        d, T, m = case["d_model"], case["seq"], _masked(case)
        block = 4 * d * d + 2 * d * case["ffn"] + 2 * T * d       # Linear layers and the two attention products, per token
        flops = 6 * B * (T * case["layers"] * block + m * d * case["vocab"])
        nbytes += B * (T + 2 * m) * 4
    else:
        c, hw = case["width"], case["img"] * case["img"]
        first = 9 * case["in_ch"] * c
        flops = 2 * B * hw * (2 * first + 3 * 2 * case["blocks"] * 9 * c * c) + 6 * B * c * case["classes"]
        nbytes += B * (hw * case["in_ch"] * 2 + 4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what was measured after one and after two steps, over these cases and drawn ones, between the
    step and the same step in float64 (with its operands rounded alike) or with the sums of its products in another
    order.  The outputs are parameters, of which a step changes 1e-4 to 2e-2, so these figures are small:

      fp32 MLP       3e-8, the rounding of the updated parameters themselves (2e-7 for one entry)
      bf16 MLP       1e-5 at width 4096 and three hidden layers, more on narrow and deep ones: a last-bit difference of a
                     pre-activation flips bf16 roundings of the activation, and layer by layer the runs drift apart
                     (1e-5 at width 8192 and six layers, 6e-5 at 1104 and six; 1e-3 for one entry)
      conv           2e-6, and 4e-5 with three blocks (7e-4 for one entry)
      encoder        3e-6 in fp32, 1e-4 in bf16.  Adam's first steps are lr times the SIGN of the gradient, so an entry
                     whose gradient is within rounding of zero (the key biases: exactly zero) moves either way
                     (two steps of 2 lr: 8e-3 of the parameters' rms)
    """
    if case["kind"] == "encoder":
        return {"rel": 4e-4 if case["dtype"] == "bf16" else 2e-5, "max": 2.5e-2}
    if case["kind"] == "conv":
        return {"rel": 2e-5 if case["blocks"] < 3 else 2e-4, "max": 3e-3}
    if case["dtype"] == "f32":
        return {"rel": 4e-7, "max": 2e-5}
    hidden = _dims(case)[1:-1]
    return {"rel": 0.16 * len(hidden) / sum(hidden) * max(1.0, len(hidden) / 3.0), "max": 4e-3}
