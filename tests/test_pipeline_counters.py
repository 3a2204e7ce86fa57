"""Host side of DeltaPipeline's calls, without a device: which counters a step
clears when the caller has put memory of its own in their place."""
import types

import torch

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
