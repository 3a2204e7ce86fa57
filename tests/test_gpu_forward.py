"""dte_adamw_forward against the oracle at the edges of its kernels: partial
float4 quads and blocks, bases at every element alignment, neighbours of the
range untouched, and sizes on both sides of the line above which the step
goes past the caches."""
import numpy as np
import pytest
import torch

from oracle import core as ocore
from paper_2608_00455_amd import binding as B
from synth import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [W.ORDER_FOLDED, W.ORDER_LITERAL])
@pytest.mark.parametrize("n", [1, 3, 4, 1023, 1024, 1026, 5 * 1024 + 7, 1 << 24, (1 << 24) + 3])
def test_forward_edges(n, order):
    hp = W.StepHP(lr=1e-4, weight_decay=0.1, order=order)
    sc = ocore.derive_scalars(hp)
    rng = np.random.default_rng(n)
    full = n + 8
    x = [rng.standard_normal(full, dtype=np.float32) * np.float32(s)
         for s in (0.02, 1e-4, 1e-6, 1e-3)]
    x[2] = np.abs(x[2])
    for off in (0, 1, 2, 3) if n < 1 << 20 else (0, 3):
        print("case: forward n %d offset %d order %d" % (n, off, order), flush=True)
        d = [torch.from_numpy(a).cuda() for a in x]
        B.dte_adamw_forward(*(t.data_ptr() + 4 * off for t in d), n, hp,
                            torch.cuda.current_stream().cuda_stream)
        want = ocore.adamw_forward(*(a[off:off + n] for a in x), sc)
        for t, a, w in zip(d, x, want):
            a = a.copy()
            a[off:off + n] = w
            assert np.array_equal(t.cpu().numpy().view(np.uint32), a.view(np.uint32))
