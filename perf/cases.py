"""The training iterations whose speed this repository is judged by, each as one case.

A pass is what a user's training loop does for one batch: `train_step` on host token and label
arrays (plan lookup, forward, loss, backward with the layers the plan rebuilds), and then
`optimizer_step` where the case updates the parameters.  The models, batch sizes, length ranges and
memory budgets are those of `synthdata.WORKLOADS`; batch sizes and lengths of padded batches also
follow the fine-tuning tasks those workloads stand for (sequences of 35-141, 153-512 and 30-332
tokens, batches of 12, 16 and 32).

Fields of a case
  model     entry of synthdata.WORKLOADS: shape and budget fraction
  dtype     storage type, "bf16" or "fp32"
  batch, length   the batch's tensor is [batch, length]
  shortest  0: every sample has `length` tokens; else the batch is padded and its samples have
            evenly spread lengths from `shortest` to `length`, in an order drawn from the seed
  dropout   probability at every site, 0 = off
  update    whether the pass ends with the AdamW update
  wait      whether the loop reads the loss after every iteration, or queues the iterations
"""
import numpy as np
import torch

import paper_2209_02478_amd as mi
import synthdata

ADAMW = dict(lr=1e-5, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)


def _case(name, model, dtype, batch, length, shortest=0, dropout=0.0, update=True, wait=False):
    return {"name": name, "model": model, "dtype": dtype, "batch": batch, "length": length, "shortest": shortest,
            "dropout": dropout, "update": update, "wait": wait}


def listed():
    return [
        # the smallest configuration: launches and latency, the loss read every time
        _case("tiny_fp32", "tiny", "fp32", 4, 33, wait=True),
        # a handful of short sequences through a real model (small per-device batches)
        _case("bert_base_b2_odd", "bert_base", "bf16", 2, 37),
        # the headline workload: a short batch, its median batch, its longest (rebuilds layers)
        _case("bert_base_short", "bert_base", "bf16", 32, 88),
        _case("bert_base_median", "bert_base", "bf16", 32, 200),
        _case("bert_base_longest", "bert_base", "bf16", 32, 512),
        # fine-tuning on question answering: padded batch of 12, dropout on, loss logged every step
        _case("bert_base_finetune", "bert_base", "bf16", 12, 397, shortest=153, dropout=0.1, wait=True),
        # multiple choice in full precision: padded batch of 16 short samples
        _case("bert_base_fp32", "bert_base", "fp32", 16, 141, shortest=35),
        # sentence pairs: padded batch of 32 through layers of three widths
        _case("bert_stages_padded", "bert_stages", "bf16", 32, 332, shortest=30),
        # the larger encoder at its middle length, forward and backward alone
        _case("bert_large_middle", "bert_large", "bf16", 64, 320, update=False),
        # causal decoder, pre-LN: median (odd) and longest context
        _case("gpt2_median", "gpt2_medium", "bf16", 16, 397),
        _case("gpt2_longest", "gpt2_medium", "bf16", 16, 1024),
        # the largest: 131072 tokens under a tight budget
        _case("bert_large_stress", "bert_large_stress", "bf16", 256, 512),
    ]


# model, dtype, batch range, length range
RANGES = [
    ("tiny", "fp32", 1, 8, 8, 64),
    ("bert_base", "bf16", 1, 32, 16, 512),
    ("bert_base", "bf16", 12, 32, 64, 512),
    ("bert_base", "fp32", 1, 16, 16, 256),
    ("bert_stages", "bf16", 4, 32, 32, 512),
    ("bert_large", "bf16", 4, 64, 32, 512),
    ("gpt2_medium", "bf16", 1, 16, 64, 1024),
    ("bert_large_stress", "bf16", 64, 256, 32, 512),
]


def draw(rng):
    model, dtype, b0, b1, l0, l1 = rng.choice(RANGES)
    spread = lambda lo, hi: min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))  # noqa: E731
    batch, length = spread(b0, b1), spread(l0, l1)
    # dropout only where the pass stays below the largest listed case
    drop = rng.random() < 0.25 and batch * length <= 1 << 16
    c = _case("", model, dtype, batch, length,
              shortest=max(1, round(length * rng.uniform(0.1, 0.8))) if rng.random() < 0.3 else 0,
              dropout=0.1 if drop else 0.0, update=rng.random() < 0.8, wait=rng.random() < 0.3)
    del c["name"]
    return c


def _shape(case):
    d = synthdata.shape_dict(synthdata.WORKLOADS[case["model"]].shape)
    d["dtype"] = case["dtype"]
    return synthdata.ModelShape(**d)


def _lengths(case):
    return np.round(np.linspace(case["shortest"], case["length"], case["batch"])).astype(np.int32) if case["batch"] > 1 \
        else np.array([case["length"]], dtype=np.int32)


def _budget(case, shape):
    """The workload's fraction of the peak without checkpointing at the longest input; small batches,
    whose memory is mostly parameters, get what keeping the boundary tensors alone needs."""
    cal = mi.Mimose(synthdata.shape_dict(shape), 0, device=None)
    if case["update"]:
        cal.optimizer_init(**ADAMW)
    cal.force_plan(0)
    none, _ = cal.dry_step(case["batch"], shape.max_seq)
    cal.force_plan((1 << shape.n_layers) - 1)
    every, _ = cal.dry_step(case["batch"], shape.max_seq)
    cal.close()
    return max(int(none * synthdata.WORKLOADS[case["model"]].budget_frac), every + every // 64 + (1 << 20))


class _State:
    pass


def prepare(case, seed):
    """A context past its data-collecting phase, with loaded weights, and one host batch."""
    shape = _shape(case)
    s = _State()
    s.update, s.wait = case["update"], case["wait"]
    s.m = m = mi.Mimose(synthdata.shape_dict(shape), _budget(case, shape))
    base = -m.arena.data_ptr() % 256

    # the context's own device buffers: parameters, gradients, and with the update its state (two
    # moments of each tensor, and the fp32 master copy of a bf16 model), each tensor on 256 bytes
    counts = [int(np.prod(m.shapes[n])) for n in m.names]
    up = lambda nbytes: (nbytes + 255) // 256 * 256  # noqa: E731
    es = 2 if case["dtype"] == "bf16" else 4
    n_params, n_grads = sum(up(n * es) for n in counts), sum(up(n * 4) for n in counts)
    part = lambda at, nbytes, dtype: m.arena[base + at:base + at + nbytes].view(dtype)  # noqa: E731
    s.outputs = {"params": part(0, n_params, torch.bfloat16 if es == 2 else torch.float32)}
    s.outputs["params"].zero_()            # the gaps between tensors too
    if case["update"]:
        s.outputs["state"] = part(n_params + n_grads, (3 if es == 2 else 2) * n_grads, torch.float32)
    # gradients by kind of tensor (their sizes differ by orders of magnitude): one output for each
    # run of layers of one width, one for each tensor outside the layers
    grads, at, runs = part(n_params, n_grads, torch.float32), 0, {}
    for name, n in zip(m.names, counts):
        kind = name
        if name.startswith("layer"):
            layer, kind = name.split(".")
            kind = "layers_%d.%s" % (shape.ffn_of(int(layer[5:])), kind)
        runs.setdefault(kind, []).append((at, n))
        at += up(n * 4) // 4
    for kind, where in runs.items():
        (at, n), pitch = where[0], where[1][0] - where[0][0] if len(where) > 1 else 1
        s.outputs["grad." + kind] = grads.as_strided((len(where), n), (pitch, 1), grads.storage_offset() + at)

    g = torch.Generator(device="cuda").manual_seed(seed)
    pool = (torch.randn(sum(counts), generator=g, device="cuda") * 0.02).cpu().numpy()
    params, at = {}, 0
    for name, shp, kind in synthdata.param_shapes(shape):
        n = int(np.prod(shp))
        params[name] = pool[at:at + n].reshape(shp) if kind == "normal" else \
            np.full(shp, 1.0 if kind == "ones" else 0.0, dtype=np.float32)
        at += n
    m.load_params(params)
    if case["update"]:
        m.optimizer_init(**ADAMW)
    if case["dropout"]:
        m.set_dropout(case["dropout"], case["dropout"], seed=seed)
    for k in range(10):                    # the collecting phase, on the allocator's bookkeeping alone
        m.dry_step(case["batch"], max(1, shape.max_seq * (k % 5 + 1) // 5))
    s.lengths = None
    if case["shortest"]:
        lengths = np.random.Generator(np.random.PCG64(seed)).permutation(_lengths(case))
        s.tokens, s.labels, s.lengths = synthdata.make_padded_batch(shape, lengths, seed)
    else:
        s.tokens, s.labels = synthdata.make_batch(shape, case["batch"], case["length"], seed)
    return s


def run(s):
    loss, _, _ = s.m.train_step(s.tokens, s.labels, s.lengths, wait=s.wait)
    if s.update:
        s.m.optimizer_step()
    return dict(s.outputs, loss=loss) if s.wait else s.outputs


def work(case):
    """Bytes: parameters read, gradients written; with the update moments and master values read and
    written and the parameters written; ids and labels.  Operations: the products of forward and
    backward over the real tokens, nothing for rebuilt layers."""
    shape = _shape(case)
    es = 2 if case["dtype"] == "bf16" else 4
    n = sum(int(np.prod(shp)) for _, shp, _ in synthdata.param_shapes(shape))
    nbytes = n * (es + 4) + case["batch"] * case["length"] * 8
    if case["update"]:
        nbytes += n * (16 + (8 if es == 2 else 0) + es)
    lengths = _lengths(case) if case["shortest"] else np.full(case["batch"], case["length"])
    tokens, pairs = float(lengths.sum()), float((lengths.astype(np.float64) ** 2).sum())
    H, V = shape.hidden, shape.vocab
    dense = sum(8.0 * H * H + 4.0 * H * shape.ffn_of(l) for l in range(shape.n_layers))
    head = 2.0 * H * V + (2.0 * H * H if shape.head else 0.0)
    attn = 4.0 * H * shape.n_layers * (0.5 if shape.causal else 1.0)
    return {"bytes": nbytes, "flops": 3.0 * (tokens * (dense + head) + pairs * attn)}


def tolerance(case):
    """Gradients pass through up to 24 layers of roundings to the storage type: in bf16 every kind of
    tensor is then 1-2 % from its fp32 value, and an element that is a long sum with cancellation is
    off by a good part of its tensor's root mean square."""
    return {"rel": 2e-2, "max": 0.9} if case["dtype"] == "bf16" else {"rel": 1e-4, "max": 1e-2}
