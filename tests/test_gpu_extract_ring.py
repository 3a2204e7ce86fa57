"""The extract kernel's stream of 256-element slots against the oracle where
its shapes can go wrong: ranges just below, at and above whole slots, whole
rings (two slots in flight per wave), whole tiles of eight slots and whole
blocks of waves, ranges that give every wave an odd or an even number of
slots, bases at every element alignment, sparse deltas and ones that select
every element of a slot (the candidate queue and the staging area at their
fullest), and decay factors below, at and above one (the bound of theta_hat
differs)."""
import sys

import numpy as np
import pytest
import torch

from oracle import core as ocore
from paper_2608_00455_amd import binding as B
from synth import workloads as W

pytestmark = pytest.mark.gpu

SLOT, RING, TILE, WAVES = 256, 2 * 256, 8 * 256, 12
# up to four slots per wave blocks are added (of 256 CUs, one block each), then
# the waves' ranges grow: 5, 6 and 9 slots each
SIZES = [3, SLOT - 1, SLOT, SLOT + 1, RING - 1, RING, RING + 5, TILE - 1, TILE + 5,
         WAVES * 4 * SLOT - 2, WAVES * 4 * SLOT + 1, WAVES * TILE * 5 + 3,
         256 * WAVES * 5 * SLOT, 256 * WAVES * 5 * SLOT + 9 * SLOT + 7, 256 * WAVES * 9 * SLOT + 7]


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def state(n, seed, hp):
    rng = np.random.default_rng(seed)
    z = lambda s: (rng.standard_normal(n, dtype=np.float32) * np.float32(s))  # noqa: E731
    return ocore.adamw_forward(z(0.02), z(1e-4), np.abs(z(1e-6)), z(1e-3),
                               ocore.derive_scalars(hp))


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("lr,wd", [(1e-5, 0.01), (1e-4, -0.05), (1e-2, 0.0), (0.3, 0.5)])
def test_slots_rings_and_alignments(n, lr, wd):
    hp = W.StepHP(lr=lr, weight_decay=wd)
    sc = ocore.derive_scalars(hp)
    p, m, v = state(n + 3, n, hp)
    dp, dm, dv = (torch.from_numpy(x).cuda() for x in (p, m, v))
    for off in ((0, 1, 2, 3) if n < 1 << 20 else (0, 3)):
        want_i, want_v, want_ph = ocore.detect(p[off:off + n], m[off:off + n], v[off:off + n], sc,
                                               off)
        for with_prev in (False, True):
            say("case: slots n %d lr %g wd %g offset %d prev %d" % (n, lr, wd, off, with_prev))
            idx = torch.full((n,), -1, dtype=torch.int64, device="cuda")
            val = torch.zeros(n, dtype=torch.int16, device="cuda")
            cur = torch.zeros(1, dtype=torch.int64, device="cuda")
            prev = torch.zeros(n + 3, dtype=torch.float32, device="cuda")
            at = lambda t: t.data_ptr() + 4 * off  # noqa: E731
            B.dte_extract_delta(at(dp), at(dm), at(dv), n, off, hp, idx.data_ptr(),
                                val.data_ptr(), n, cur.data_ptr(), at(prev) if with_prev else 0,
                                torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            k = int(cur.item())
            assert k == want_i.size
            got = idx[:k].cpu().numpy()
            o = np.argsort(got)
            assert np.array_equal(got[o], want_i)
            assert np.array_equal(val[:k].cpu().numpy().view(np.uint16)[o], want_v)
            if with_prev:
                out = prev.cpu().numpy().view(np.uint32)
                assert np.array_equal(out[off:off + n], want_ph.view(np.uint32))
                assert not out[:off].any() and not out[off + n:].any()
