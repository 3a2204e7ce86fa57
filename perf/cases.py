"""Benchmark cases: the calls a user of this framework makes, through its
public entry points, over the range of sizes and options it supports.

A case names a model shape, a trainer layout, a receiver layout, a step size
and a call:

  step      DeltaPipeline.step: reset, extract, remap, apply (with
            parameter groups when the norms take no weight decay: one
            extract call per run of equal step scalars);
  fused     DeltaPipeline.step_fused: detection and remap in one pass;
  ordered   DeltaPipeline.step with the delta in ascending offset order;
  prev      DeltaPipeline.extract with theta_hat requested, ordered delta;
  forward   dte_adamw_forward, the trainer-side step that extract inverts;
  publish   the storage path: an ordered delta written from the device,
            committed, read back into device memory, remapped and applied.

States are the seeded synthetic ones of `synth` (Irwin-Hall weights of
sigma 0.02, one AdamW step on the device); the receivers' previous weights
are random BF16 of the same scale.  All results are bit patterns, counts or
correctly rounded binary32 values, so every tolerance is "exact".
"""
import math
import os
import tempfile
from dataclasses import replace

import torch

import synth
from paper_2608_00455_amd import binding as B
from paper_2608_00455_amd import store as S
from paper_2608_00455_amd.layouts import build_spec, sender_segments, store_pieces
from paper_2608_00455_amd.pipeline import DeltaPipeline, generate_state, group_runs
from synth import workloads as W

# Qwen3-8B and the tiny block, per-layer shapes as in synth.workloads
QWEN8B = dict(hidden=4096, heads_q=32, heads_kv=8, head_dim=128, intermediate=12288)
SMALL = dict(hidden=256, heads_q=4, heads_kv=2, head_dim=64, intermediate=704)


def listed():
    return [
        # the smallest model of the tests (2 layers with embeddings): a step
        # that is nothing but launches and latency
        dict(name="step_small", call="step", model="dense", layers=2, vocab=1000, tp=2, lr=1e-6,
             **SMALL),
        # one dense block of 11 M elements: a block-wise or pipelined sync
        dict(name="step_tiny_block", call="step", model="tiny", tp=2, lr=1e-6),
        # odd hidden size, norms in a group without decay: tensors and
        # extract ranges begin at odd offsets
        dict(name="step_odd_groups", call="step", model="dense", layers=3, vocab=6002, tp=2,
             lr=1e-4, hidden=1001, heads_q=8, heads_kv=2, head_dim=128, intermediate=2730,
             groups=True),
        # four Qwen3-8B layers: one pipeline stage's shard at an RL step size
        dict(name="step_4l", call="step", model="dense", layers=4, vocab=0, tp=4, lr=1e-6,
             **QWEN8B),
        # the same at a pre-training step size (14 % of the weights change),
        # norms without weight decay: many extract calls, a dense delta
        dict(name="step_4l_dense_groups", call="step", model="dense", layers=4, vocab=0, tp=4,
             lr=1e-4, groups=True, **QWEN8B),
        # mixture of experts: Qwen3-30B-A3B layers on eight receivers, most
        # experts untouched, router and norms replicated
        dict(name="step_moe_ep8", call="step", model="moe30b", layers=2, lr=1e-5),
        # the largest: sixteen Qwen3-8B layers (3.1e9 elements), TP=8
        dict(name="step_16l_tp8", call="step", model="dense", layers=16, vocab=0, tp=8, lr=1e-6,
             **QWEN8B),
        # a Megatron-Core trainer shard with the ordered delta that the
        # sparse payload of a sender-receiver pair asks for
        dict(name="ordered_mcore", call="ordered", model="mcore", layers=4, vocab=0, trainer_tp=2,
             trainer_rank=1, tp=4, lr=1e-5, **QWEN8B),
        # detection and remap in one pass
        dict(name="fused_2l", call="fused", model="dense", layers=2, vocab=0, tp=4, lr=1e-5,
             **QWEN8B),
        # the reconstructed master weights themselves (checks, checkpoints),
        # in the operation order of the printed inverse
        dict(name="prev_literal_1l", call="prev", model="dense", layers=1, vocab=0, tp=4, lr=1e-6,
             order=W.ORDER_LITERAL, **QWEN8B),
        # the trainer's own AdamW step
        dict(name="forward_1l", call="forward", model="dense", layers=1, vocab=0, tp=4, lr=1e-6,
             **QWEN8B),
        # storage-mediated publication to another cluster and back
        dict(name="publish_tiny", call="publish", model="tiny", tp=2, lr=1e-5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same calls and options: 3e5 to 6e8 elements (storage
    path: 1e6 to 1e7), odd sizes among them, step sizes of 1e-7 to 1e-4
    (storage path: 1e-6 to 1e-5), one to eight receivers."""
    call = rng.choice(["step", "step", "step", "step", "fused", "ordered", "prev", "forward",
                       "publish"])
    model = rng.choice(["dense", "dense", "mcore", "moe"])
    least, most, slow, fast = (1e6, 1e7, -6, -5) if call == "publish" else (3e5, 6e8, -7, -4)
    numel = math.exp(rng.uniform(math.log(least), math.log(most)))
    c = dict(call=call, model=model, lr=10.0 ** rng.uniform(slow, fast),
             order=rng.choice([W.ORDER_FOLDED, W.ORDER_FOLDED, W.ORDER_LITERAL]),
             groups=call in ("step", "ordered", "fused") and rng.random() < 0.3)
    # about 12.5 hidden^2 elements per dense layer: hidden follows from the
    # drawn size
    layers = rng.randint(1, 4)
    hidden = max(96, min(6144, int(math.sqrt(numel / (12.5 * layers)))))
    hidden = hidden if rng.random() < 0.4 else hidden // 64 * 64
    tp = rng.choice([1, 2, 4, 8])
    head_dim = rng.choice([32, 64, 128])
    kv = 8
    heads = kv * max(1, round(hidden / (kv * head_dim)))
    inter = 8 * max(1, int(hidden * rng.uniform(2.5, 3.5)) // 8)
    if model == "moe":
        ranks = rng.choice([2, 4, 8])
        experts = ranks * rng.choice([2, 4])
        width = max(8, int(numel / (3.0 * layers * experts * hidden)))
        c.update(layers=layers, ranks=ranks, attn_tp=rng.choice([1, 2]), experts=experts,
                 hidden=hidden, heads_q=heads, heads_kv=kv, head_dim=head_dim,
                 expert_intermediate=min(width, 2 * hidden))
        return c
    vocab = 8 * _log_int(rng, 64, 2048) if rng.random() < 0.5 else 0
    c.update(layers=layers, vocab=vocab, tp=tp, hidden=hidden, heads_q=heads, heads_kv=kv,
             head_dim=head_dim, intermediate=inter)
    if model == "mcore":
        c.update(trainer_tp=2, trainer_rank=rng.randint(0, 1))
    return c


def _workload(case, seed):
    shape = {k: case[k] for k in ("layers", "hidden", "heads_q", "heads_kv", "head_dim",
                                  "intermediate", "vocab", "experts", "expert_intermediate",
                                  "ranks", "attn_tp") if k in case}
    model = case["model"]
    if model == "tiny":
        wl = W.tiny_block()
    elif model == "moe30b":
        wl = W.qwen3_30b_a3b_share(synth.word, layers=case["layers"])
    elif model == "moe":
        wl = W.scaled_moe(synth.word, **shape)
    elif model == "mcore":
        wl = W.scaled_mcore(trainer_tp=case["trainer_tp"], trainer_rank=case["trainer_rank"],
                            receiver_tp=case["tp"], **shape)
    else:
        wl = W.scaled_dense(tp=case["tp"], embed=case["vocab"] > 0, **shape)
    hp = replace(wl.hp, lr=case["lr"], order=case.get("order", W.ORDER_FOLDED))
    wl = replace(wl, seed=W.SEED_BASE + 1009 * int(seed), hp=hp)
    return W.with_norm_group(wl) if case.get("groups") else wl


def _numel(case):
    return sum(math.prod(s.shape) for s in sender_segments(_workload(case, 0)))


# share of the elements whose BF16 pattern changes under the synthetic
# recipe, by learning rate (weights of untouched experts change none)
_CHANGE = ((1e-7, 0.000403), (1e-6, 0.00317), (1e-5, 0.0227), (1e-4, 0.138))


def _change_fraction(lr):
    x = math.log10(lr)
    for (l0, f0), (l1, f1) in zip(_CHANGE, _CHANGE[1:]):
        if lr <= l1 * 1.0001:
            w = (x - math.log10(l0)) / (math.log10(l1) - math.log10(l0))
            return math.exp(math.log(f0) * (1 - w) + math.log(f1) * w)
    return _CHANGE[-1][1]


class _Scratch:
    """A store directory in memory-backed storage, removed with the state."""

    def __init__(self):
        base = "/dev/shm" if os.path.isdir("/dev/shm") else None
        self.dir = tempfile.TemporaryDirectory(prefix="dte_store_", dir=base)

    @property
    def path(self):
        return self.dir.name


def prepare(case, seed):
    wl = _workload(case, seed)
    call = case["call"]
    st = dict(case=case, wl=wl, hp=wl.hp)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    if call == "forward":
        p, m, v = generate_state(wl)
        g = torch.randn(p.numel(), generator=gen, device="cuda").mul_(1e-3)
        st.update(p=p, m=m, v=v, g=g)
        return st
    spec = build_spec(wl)
    n = spec.total
    # room for half as many changes again as the step size makes expect, and
    # at least 2 % of the shard
    capacity = int(n * max(0.02, 1.5 * _change_fraction(case["lr"]))) + 4096
    shards = None
    if call != "prev":
        shards = []
        for k in spec.rank_numel:
            t = torch.empty(k, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02,
                                                                            generator=gen)
            shards.append(t.view(torch.int16))
    pipe = DeltaPipeline(spec, capacity, shards=shards,
                         ordered=call in ("ordered", "prev", "publish"),
                         rank_capacity=[1] * spec.nranks if call == "prev" else None)
    pipe.idx.zero_()   # an ordered delta is returned whole: nothing beyond its end
    pipe.val.zero_()
    p, m, v = generate_state(wl)
    runs = group_runs(wl)
    st.update(pipe=pipe, p=p, m=m, v=v, runs=runs if len(runs) > 1 else None)
    if call == "prev":
        st["prev"] = torch.empty(n, dtype=torch.float32, device="cuda")
    if call == "publish":
        st["segs"] = S.segments_of([t.name for t in wl.tensors], wl.flat_begins(),
                                   [t.numel for t in wl.tensors])
        st["pieces"] = (S.pieces_of(store_pieces(wl)) if wl.sender.kind == "mcore" else None)
        st["scratch"] = _Scratch()
        # the receiving side: the canonical tensors into the same receivers
        dst_wl = W.canonical_twin(wl) if wl.sender.kind == "mcore" else wl
        dst_spec = build_spec(dst_wl)
        st["dst"] = DeltaPipeline(dst_spec, capacity, shards=shards)
        pipe.reset()
        pipe.extract_runs(p, m, v, runs)
        torch.cuda.synchronize()
    return st


def run(st):
    call = st["case"]["call"]
    if call == "forward":
        s = torch.cuda.current_stream().cuda_stream
        B.dte_adamw_forward(st["p"].data_ptr(), st["m"].data_ptr(), st["v"].data_ptr(),
                            st["g"].data_ptr(), st["p"].numel(), st["hp"], s)
        return {"p": st["p"], "m": st["m"], "v": st["v"]}
    pipe, p, m, v, hp = st["pipe"], st["p"], st["m"], st["v"], st["hp"]
    if call == "step":
        pipe.step(p, m, v, hp, runs=st["runs"])
    elif call == "fused":
        pipe.step_fused(p, m, v, hp, runs=st["runs"])
    elif call == "ordered":
        pipe.step(p, m, v, hp, runs=st["runs"])
        return {"idx": pipe.idx, "val": pipe.val, "count": pipe.cursor,
                "rank_count": pipe.rank_count, "shards": pipe.shards}
    elif call == "prev":
        pipe.reset()
        pipe.extract(p, m, v, hp, out_prev=st["prev"])
        return {"prev": st["prev"], "idx": pipe.idx, "val": pipe.val, "count": pipe.cursor}
    elif call == "publish":
        return _publish(st)
    return {"count": pipe.cursor, "rank_count": pipe.rank_count, "shards": pipe.shards}


def _publish(st):
    pipe, dst, path = st["pipe"], st["dst"], st["scratch"].path
    s = torch.cuda.current_stream().cuda_stream
    S.write_part_device(path, 1, 0, st["segs"], pipe.idx.data_ptr(), pipe.val.data_ptr(),
                        pipe.cursor.data_ptr(), pipe.capacity, stream=s, pieces=st["pieces"])
    S.commit(path, 1, 0, 1)
    n, _ = S.read_device(path, 1, 0, dst.idx.data_ptr(), dst.val.data_ptr(), dst.capacity, stream=s)
    dst.cursor.fill_(n)
    dst.remap()
    dst.apply()
    return {"count": dst.cursor, "rank_count": dst.rank_count, "shards": dst.shards}


def work(case):
    """One pass's unavoidable bytes: the step reads theta, m, v (12 bytes an
    element) and writes the delta (10 bytes an entry), the buckets (10) and
    the receivers' new values (2); the fused step writes no delta."""
    n = _numel(case)
    wl = _workload(case, 0)
    touched = sum(t.numel for t in wl.tensors if t.touched) / max(1, wl.numel)
    entries = n * _change_fraction(case["lr"]) * touched
    call = case["call"]
    if call == "forward":
        return {"bytes": 28.0 * n, "flops": 14.0 * n}
    if call == "prev":
        return {"bytes": 16.0 * n + 10.0 * entries, "flops": 8.0 * n}
    if call == "publish":   # delta read, stored (6 bytes an entry), read back, routed, applied
        return {"bytes": (10 + 6 + 6 + 10 + 10 + 2) * entries, "flops": 1.0 * entries}
    per_entry = 12 if call == "fused" else 22
    return {"bytes": 12.0 * n + per_entry * entries, "flops": 8.0 * n}


def tolerance(case):
    # one rounding sequence is specified for every output: bit patterns
    return "exact"


def exact(case, seed):
    """The binary32 outputs (theta_hat; the forward step's p, m, v) in
    binary64, from the hyperparameters; bit patterns and counts have no such
    value."""
    call = case["call"]
    if call not in ("prev", "forward"):
        return None
    st = prepare(case, seed)
    hp = st["hp"]
    bc1, bc2 = 1.0 - hp.beta1 ** hp.step, 1.0 - hp.beta2 ** hp.step
    n = st["p"].numel()
    outs = {k: torch.empty(n, dtype=torch.float64, device="cuda")
            for k in (("prev",) if call == "prev" else ("p", "m", "v"))}
    part = 1 << 26
    for b in range(0, n, part):
        p, m, v = (st[k][b:b + part].double() for k in ("p", "m", "v"))
        if call == "forward":
            g = st["g"][b:b + part].double()
            m = hp.beta1 * m + (1.0 - hp.beta1) * g
            v = hp.beta2 * v + (1.0 - hp.beta2) * g * g
        u = hp.lr * (m / bc1) / ((v / bc2).sqrt() + hp.eps)
        if call == "prev":
            outs["prev"][b:b + part] = (p + u) / (1.0 - hp.lr * hp.weight_decay)
        else:
            outs["p"][b:b + part] = (1.0 - hp.lr * hp.weight_decay) * p - u
            outs["m"][b:b + part] = m
            outs["v"][b:b + part] = v
    return {"prev": outs["prev"], "idx": None, "val": None, "count": None} if call == "prev" else outs
