"""The queue cache's extension in the state buffer (kernels for more than 64
instances) at less than one entry per slot, as in handles whose extension the
state buffer's budget cuts: full extensions drop entries and take no more.
Bit-exact against the oracle; the kept order must never change a result."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import preset  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU-only hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_16336_amd import Scheduler  # noqa: E402
from paper_2608_16336_amd.mts import MtsError  # noqa: E402


def _cfg(I, S, M, arrival, R=2, K=10, interval=1, out=40.0, **kw):
    c = preset("tiny")
    c.update(n_instances=I, slots_per_instance=S, kv_blocks=M, headroom_base=M / 8.0, headroom_decay=0.7, mig_interval=interval,
             mig_max_pairs=I // 2, mig_stage_blocks=4, arrival=arrival, prompt=dict(kind="uniform_int", lo=16, hi=600),
             output=dict(kind="geometric", mean=out), groups=[dict(n_replicas=R, K=K, tiers=dict(kind="uniform"))], seed=31)
    c.update(kw)
    return c


def _same(g, o, what):
    got, want = g.export(), o.export()
    for k in want:
        assert np.array_equal(got[k], want[k]), "%s: field %s" % (what, k)


def test_the_depth_in_use_is_lowered_and_raised_between_steps():
    cfg = _cfg(130, 256, 300, dict(kind="gamma_poisson", mean=120.0, cv=3.0))
    g, o = Scheduler(cfg), oracle.Oracle(cfg)
    assert g.queue_extension() == (256, 256)
    for depth in (63, 257, 0):
        with pytest.raises(MtsError) as e:
            g.set_queue_extension(depth)
        assert e.value.code == -1
    for depth, ticks in ((256, 40), (64, 30), (65, 1), (200, 17), (64, 30), (256, 10)):
        g.set_queue_extension(depth)
        assert g.queue_extension() == (depth, 256)
        g.step(ticks)
        o.step(ticks)
        _same(g, o, "depth %d" % depth)
    assert g.stats()["raw"][86] == 0
    g = Scheduler(_cfg(64, 64, 300, dict(kind="poisson", mean=9.0)))
    assert g.queue_extension() == (0, 0)
    with pytest.raises(MtsError):
        g.set_queue_extension(64)
