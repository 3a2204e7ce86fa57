"""dte_extract_runs and the one-pass step over runs against the oracle, run by
run: runs that begin and end inside a slot, several of them in one slot, one
element long, empty, more than one launch takes, gaps between runs, changes
of the operation order and of the decay factor (below, at and above one), runs
in the dynamic tail and runs long enough for a launch of their own between
short ones, in both output orders, with and without theta_hat."""
import numpy as np
import pytest
import torch

from oracle import core as ocore
from paper_2608_00455_amd import binding as B
from paper_2608_00455_amd import layouts
from paper_2608_00455_amd.pipeline import DeltaPipeline
from synth import workloads as W

pytestmark = pytest.mark.gpu

HPS = [W.StepHP(lr=1e-4, weight_decay=0.01), W.StepHP(lr=1e-4, weight_decay=0.0),
       W.StepHP(lr=1e-2, weight_decay=-0.05), W.StepHP(lr=1e-3, weight_decay=0.3, step=7)]
LITERAL = W.StepHP(lr=1e-4, weight_decay=0.01, order=W.ORDER_LITERAL)


def cuts(kind, n, rng):
    """Run boundaries of [0, n)."""
    if kind == "slots":            # whole slots and blocks of waves
        return [0, 256, 512, 12 * 4 * 256, n]
    if kind == "tiny":             # several runs per slot, one-element and empty runs
        return [0, 1, 2, 2, 5, 200, 255, 256, 257, 300, 300, 301, 700, n - 1, n]
    if kind == "many":             # more runs than one launch takes
        return [0] + sorted(int(x) for x in rng.integers(1, n, 75)) + [n]
    if kind == "split":            # a run of 2^24 elements and more between short ones
        return [0, 5001, 5001 + (1 << 24) + 333, n - 901, n]
    # "tail": runs that begin in the dynamic tail (the last 1/16 of the slots):
    # just before it, inside slots, at a chunk of 96 slots and inside one, one
    # element long, in the partial slot at the end
    slots = (n + 255) // 256
    t, chunk = (slots - slots // 16) * 256, 96 * 256
    return [0, n // 3 | 1, 2 * (n // 3), t - 300, t + 1000, t + chunk, t + 5 * chunk + 13, t + 5 * chunk + 14,
            t + 9 * chunk + 256 * 40, n - 20, n]


def size(kind):
    if kind == "split":
        return 5001 + (1 << 24) + 333 + 700 + 901
    # the tail begins when the waves (12 per CU) have 48 slots each
    waves = 12 * torch.cuda.get_device_properties(0).multi_processor_count
    return (48 * waves + 1000) * 256 + 77


def state(n, seed):
    rng = np.random.default_rng(seed)
    z = lambda s: (rng.standard_normal(n, dtype=np.float32) * np.float32(s))  # noqa: E731
    return ocore.adamw_forward(z(0.02), z(1e-4), np.abs(z(1e-6)), z(1e-3),
                               ocore.derive_scalars(HPS[0]))


@pytest.mark.parametrize("kind,n", [("slots", 5 * 12 * 1024), ("tiny", 1003), ("tiny", 40000),
                                    ("many", 300_001), ("tail", None), ("split", None)])
@pytest.mark.parametrize("orders", ["folded", "literal", "both"])
@pytest.mark.parametrize("ordered", [False, True])
def test_runs_against_oracle(kind, n, orders, ordered):
    if n is None:
        if orders == "both" or (orders == "literal" and ordered):
            pytest.skip("covered at the small sizes")
        n = size(kind)
    print("case: runs %s n %d %s ordered %d" % (kind, n, orders, ordered), flush=True)
    rng = np.random.default_rng(n)
    at = cuts(kind, n, rng)
    hps = {"folded": HPS, "literal": [LITERAL], "both": HPS + [LITERAL]}[orders]
    if orders == "literal":
        hps = [LITERAL, W.StepHP(lr=1e-4, weight_decay=0.0, order=W.ORDER_LITERAL, eps=1e-14)]
    runs = [(b, e, hps[k % len(hps)]) for k, (b, e) in enumerate(zip(at, at[1:]))]
    if kind == "many":
        del runs[40]               # a gap
    p, m, v = state(n, n)
    want = [ocore.detect(p[b:e], m[b:e], v[b:e], ocore.derive_scalars(h), b)
            for b, e, h in runs if e > b]
    wi = np.concatenate([w[0] for w in want])
    wv = np.concatenate([w[1] for w in want])
    d = [torch.from_numpy(x).cuda() for x in (p, m, v)]
    s = torch.cuda.current_stream().cuda_stream
    for with_prev in (False, True):
        idx = torch.full((n,), -1, dtype=torch.int64, device="cuda")
        val = torch.zeros(n, dtype=torch.int16, device="cuda")
        cur = torch.zeros(1, dtype=torch.int64, device="cuda")
        prev = torch.full((n,), 7.0, dtype=torch.float32, device="cuda")
        ws = torch.empty(B.dte_ordered_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        B.dte_extract_runs(*(t.data_ptr() for t in d), runs, idx.data_ptr(), val.data_ptr(), n,
                           cur.data_ptr(), ws.data_ptr() if ordered else 0,
                           ws.numel() if ordered else 0, prev.data_ptr() if with_prev else 0, s)
        torch.cuda.synchronize()
        k = int(cur.item())
        assert k == wi.size
        gi, gv = idx[:k].cpu().numpy(), val[:k].cpu().numpy().view(np.uint16)
        if not ordered:
            o = np.argsort(gi)
            gi, gv = gi[o], gv[o]
        assert np.array_equal(gi, wi) and np.array_equal(gv, wv)
        if with_prev:
            full = np.full(n, 7.0, np.float32)
            for (b, e, _), w in zip([r for r in runs if r[1] > r[0]], want):
                full[b:e] = w[2]
            assert np.array_equal(prev.cpu().numpy().view(np.uint32), full.view(np.uint32))


@pytest.mark.parametrize("odd", [0, 3, "long"])
@pytest.mark.parametrize("order", [W.ORDER_FOLDED, W.ORDER_LITERAL])
def test_one_pass_step_over_runs(odd, order):
    """The one-pass step over runs: the same shards and buckets as the step
    ("long": a run with a launch of its own between runs that share)."""
    long = odd == "long"
    print("case: one-pass runs, odd %s order %s" % (odd, order), flush=True)
    odd = 1 if long else odd
    shape = dict(hidden=1024, heads_q=8, heads_kv=2, head_dim=128, intermediate=2816) if long \
        else dict(hidden=256 + odd)
    wl = W.scaled_dense(layers=2, tp=2, embed=False, lr=1e-4, **shape)
    spec = layouts.build_spec(wl)
    n = wl.numel
    p, m, v = (torch.from_numpy(x).cuda() for x in state(n, odd))
    hps = [W.StepHP(lr=1e-4, weight_decay=w, order=order) for w in (0.01, 0.0, -0.1)]
    at = [0, 255 + odd, 260, 300_001, 300_001 + (1 << 24) + 333, 17_100_000, n] if long else \
        [0, 255 + odd, 260, 300_001, n]
    runs = [(b, e, hps[k % 3]) for k, (b, e) in enumerate(zip(at, at[1:]))]
    pipes = [DeltaPipeline(spec, n) for _ in range(2)]
    pipes[0].step(p, m, v, None, runs=runs)
    pipes[1].step_fused(p, m, v, None, runs=runs)
    assert int(pipes[0].cursor.item()) == int(pipes[1].cursor.item()) > 0
    (b0, c0), (b1, c1) = (q.buckets() for q in pipes)
    assert np.array_equal(c0, c1)
    for r in range(len(c0)):
        assert np.array_equal(b0[r][0], b1[r][0]) and np.array_equal(b0[r][1], b1[r][1])
        assert torch.equal(pipes[0].shards[r], pipes[1].shards[r])
    # a slice of a longer state, and states that are not flat, take each run by itself
    pipes[1].reset()
    pipes[1].extract_runs(p[None], m[None], v[None], [(0, 1, hps[0])])
    with pytest.raises(ValueError):
        pipes[1].extract_runs(p, m, v, [(0, n + 1, hps[0])])
    with pytest.raises(ValueError):
        pipes[1].step_fused(p, m, v, None, runs=[(5, n + 1, hps[0])])
