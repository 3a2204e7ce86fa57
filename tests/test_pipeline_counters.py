"""Host side of DeltaPipeline's calls, without a device: which counters a step
clears when the caller has put memory of its own in their place, and which
runs its calls accept."""
import types

import pytest
import torch

from paper_2608_00455_amd import binding as B
from paper_2608_00455_amd.pipeline import DeltaPipeline


def pipeline(ranks=3):
    """The counters of a pipeline, on the CPU (no plan, no library call)."""
    q = object.__new__(DeltaPipeline)
    q.plan = types.SimpleNamespace(nranks=ranks)
    q._counters = torch.full((16 + ranks,), 7, dtype=torch.int64)
    q.cursor = q._counters[:1]
    q.rank_count = q._counters[16:]
    return q


def test_step_clears_the_counters_in_use():
    own = pipeline()
    own._reset_counters()
    assert not own.cursor.any() and not own.rank_count.any()
    for name in ("cursor", "rank_count"):
        # the tensor replaced, and the same tensor object on other memory
        for in_place in (False, True):
            q = pipeline()
            n = getattr(q, name).numel()
            other = torch.full((n,), 5, dtype=torch.int64)
            if in_place:
                getattr(q, name).set_(other)
            else:
                setattr(q, name, other)
            q._reset_counters()
            assert not other.any(), (name, in_place)
            assert not q.cursor.any() and not q.rank_count.any()
    # counters of several pipelines in one tensor: a step clears its own
    q, table = pipeline(), torch.full((8,), 5, dtype=torch.int64)
    q.rank_count = table[2:]
    q._reset_counters()
    assert table.tolist() == [5, 5, 0, 0, 0, 5, 5, 5] and not q.cursor.any()


@pytest.mark.parametrize("name", ["extract_runs", "step_fused"])
def test_runs_that_hold_no_element(monkeypatch, name):
    """An empty run is accepted wherever it lies, as the empty slice it is,
    and no runs at all need no state; a run beyond the state is refused."""
    q = pipeline()
    q.idx = torch.zeros(1, dtype=torch.int64)
    monkeypatch.setattr("paper_2608_00455_amd.pipeline._stream", lambda s=None: 0)
    q.ordered, q.workspace, q.capacity, q.val = False, None, 1, q.idx
    q.plan.handle, q.off, q.rval, q.rank_capacity, q.shards = 1, [], [], [], []
    calls = []
    for f in ("dte_extract_runs", "dte_extract_remap_apply", "dte_apply"):
        monkeypatch.setattr(B, f, lambda *a, f=f: calls.append((f, a)))
    t = torch.zeros(8)
    call = (lambda runs, x=t: q.extract_runs(x, x, x, runs)) if name == "extract_runs" else \
        (lambda runs, x=t: q.step_fused(x, x, x, None, runs=runs))
    call([(9, 9, None)])
    call([(0, 8, None), (12, 12, None)])
    call([], None)
    for run in ((0, 9, None), (9, 10, None)):
        with pytest.raises(ValueError):
            call([run])
