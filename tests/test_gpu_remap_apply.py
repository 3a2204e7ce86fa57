"""dte_remap_apply and dte_extract_remap_apply against dte_remap followed by
dte_apply: more ranks than one launch takes, buckets too small for their
entries (the shards take what the buckets took and nothing else), appended
calls on uncleared counts, and matrices, vectors and experts in one plan."""
import numpy as np
import pytest
import torch

import synth
from paper_2608_00455_amd import binding as B
from paper_2608_00455_amd.layouts import build_spec
from paper_2608_00455_amd.pipeline import DeltaPipeline, generate_state
from synth import workloads as W

pytestmark = pytest.mark.gpu

CASES = [("dense", dict(layers=2, tp=2)),
         ("dense", dict(layers=1, tp=32, heads_q=32, heads_kv=32, head_dim=8, hidden=64,
                        intermediate=1024, embed=False)),
         ("moe", dict(layers=1, ranks=4, experts=8))]


def workload(kind, kw):
    return W.scaled_moe(synth.word, lr=1e-4, **kw) if kind == "moe" else \
        W.scaled_dense(lr=1e-4, **kw)


def tensors(spec, seed):
    rng = np.random.default_rng(seed)
    return [torch.from_numpy(rng.integers(-32768, 32767, n, dtype=np.int16)).cuda()
            for n in spec.rank_numel]


def ptrs(ts):
    return [t.data_ptr() for t in ts]


@pytest.mark.parametrize("kind,kw", CASES)
@pytest.mark.parametrize("room", [1.0, 0.3, 0.0])
@pytest.mark.parametrize("fused", [False, True])
def test_shards_take_what_the_buckets_took(kind, kw, room, fused):
    print("case: remap_apply %s %s room %g fused %d" % (kind, kw, room, fused), flush=True)
    wl = workload(kind, kw)
    spec = build_spec(wl)
    if fused and len(spec.rank_numel) > 16:
        pytest.skip("the one-pass call takes at most 16 ranks")
    p, m, v = generate_state(wl)
    ref = DeltaPipeline(spec, wl.numel, shards=tensors(spec, 1))
    ref.reset()
    ref.extract(p, m, v, wl.hp)
    ref.remap()
    ref.apply()
    want, counts = ref.buckets()
    cap = [int(c * room) for c in counts]
    got = DeltaPipeline(spec, wl.numel, rank_capacity=cap, shards=tensors(spec, 1))
    for _ in range(2):          # a second step starts from cleared counts
        (got.step_fused if fused else got.step)(p, m, v, wl.hp)
    assert int(got.cursor.item()) == int(ref.cursor.item())
    have, hcounts = got.buckets()
    assert np.array_equal(hcounts, counts)
    for r, before in enumerate(tensors(spec, 1)):
        off, val = have[r]
        assert off.size == cap[r] and np.unique(off).size == off.size
        new = before.cpu().numpy().view(np.uint16)
        if room == 1.0:
            assert np.array_equal(off, want[r][0]) and np.array_equal(val, want[r][1])
            new = ref.shards[r].cpu().numpy().view(np.uint16)
        else:
            assert np.isin(off, want[r][0]).all()
        full = got.shards[r].cpu().numpy().view(np.uint16)
        if room != 0.3:
            assert np.array_equal(full, new)
        else:       # two steps took two subsets: every change is an entry's value
            at = np.flatnonzero(full != new)
            k = np.searchsorted(want[r][0], at)
            assert np.array_equal(want[r][0][k], at) and np.array_equal(want[r][1][k], full[at])
            assert np.array_equal(full[off], val)


def test_appended_calls_keep_earlier_buckets():
    wl = workload(*CASES[0])
    spec = build_spec(wl)
    p, m, v = generate_state(wl)
    ref = DeltaPipeline(spec, wl.numel, shards=tensors(spec, 2))
    ref.step(p, m, v, wl.hp)
    got = DeltaPipeline(spec, wl.numel, shards=tensors(spec, 2))
    half = wl.numel // 2 | 1
    got.cursor, got.rank_count = got.cursor.clone(), got.rank_count.clone()
    s = torch.cuda.current_stream().cuda_stream
    for b, e in ((0, half), (half, wl.numel)):
        got.reset()
        got.extract(p[b:e], m[b:e], v[b:e], wl.hp, index_base=b)
        B.dte_remap_apply(got.plan.handle, got.idx.data_ptr(), got.val.data_ptr(),
                          got.cursor.data_ptr(), got.capacity, ptrs(got.off), ptrs(got.rval),
                          got.rank_capacity, got.rank_count.data_ptr(), ptrs(got.shards), s)
    want, wc = ref.buckets()
    have, hc = got.buckets()
    assert np.array_equal(wc, hc)
    for r in range(len(wc)):
        assert np.array_equal(want[r][0], have[r][0]) and np.array_equal(want[r][1], have[r][1])
        assert torch.equal(ref.shards[r], got.shards[r])
    # counters of the caller's own are cleared as well
    got.step(p, m, v, wl.hp)
    assert np.array_equal(got.rank_count.cpu().numpy(), wc)
