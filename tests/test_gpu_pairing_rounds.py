"""Pairing rounds that can move nothing are left out (no overloaded or draining
instance holds a request, or no instance that isn't draining has a free slot);
the rounds beside them must still run.  Bit-exact against the oracle on
clusters that pass from one to the other."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import preset  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU-only hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_16336_amd import Scheduler  # noqa: E402


def _cfg(I, S, M, mean, interval=1, out=30.0):
    c = preset("tiny")
    c.update(n_instances=I, slots_per_instance=S, kv_blocks=M, headroom_base=M / 16.0, headroom_decay=0.6, mig_interval=interval,
             mig_max_pairs=I // 2, mig_stage_blocks=4, arrival=dict(kind="gamma_poisson", mean=mean, cv=1.5),
             prompt=dict(kind="uniform_int", lo=16, hi=600), output=dict(kind="geometric", mean=out),
             groups=[dict(n_replicas=2, K=4, tiers=dict(kind="uniform"))], seed=5)
    return c


@pytest.mark.parametrize("cfg", [
    # a light load: drained instances are emptied by moves and stay empty
    _cfg(9, 64, 700, 3.0),
    _cfg(64, 64, 700, 20.0, interval=3),
    # slots that run out before blocks do: full instances beside one that drains
    _cfg(7, 64, 4000, 12.0, out=60.0),
    # blocks that run out: queues to move, also onto the few with room
    _cfg(16, 64, 300, 12.0),
    _cfg(70, 64, 600, 40.0),
    _cfg(130, 64, 4000, 250.0, interval=2, out=60.0),
], ids=["light", "interval", "full_slots", "overload", "wide", "wide_full_slots"])
def test_rounds_that_move_nothing_and_rounds_that_do(cfg):
    I = cfg["n_instances"]
    g, o = Scheduler(cfg), oracle.Oracle(cfg)
    flags = np.zeros(2 * I, np.uint8)
    for ticks, drained in ((60, ()), (90, (0, 3, I - 1)), (40, (3,)), (30, range(I - 1)), (30, range(I))):
        for i in range(I):
            for r in range(2):
                o.set_drain(r, i, i in drained)
                flags[r * I + i] = i in drained
        g.set_draining(flags)
        g.step(ticks)
        o.step(ticks)
        got, want = g.export(), o.export()
        for k in want:
            assert np.array_equal(got[k], want[k]), "I=%d field %s after %d drained" % (I, k, len(drained))
    raw = want["stats"].reshape(2, -1).sum(0)
    assert raw[80] + raw[81] > 0  # requests moved, at once or by staged copies
