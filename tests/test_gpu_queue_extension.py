"""The queue cache's extension in the state buffer (kernels for more than 64
instances) at less than one entry per slot, as in handles whose extension the
state buffer's budget cuts: full extensions drop entries and take no more.
Bit-exact against the oracle; the kept order must never change a result."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import preset, with_extensions  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU-only hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_16336_amd import Scheduler  # noqa: E402
from paper_2608_16336_amd.mts import MtsError  # noqa: E402


INFAAS = dict(policy="infaas", alpha=64, beta=1, gamma=1, pen_overloaded=512, pen_interfered=128, ewma_shift=4)


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


@pytest.mark.parametrize("ring,ticks", [(1, 61), (7, 65), (15, 68)])
def test_an_arrival_that_becomes_the_head_may_push_the_extension_out(ring, ticks):
    # One instance takes every arrival (the others drain) and its queue grows
    # through the length at which head, ring and full extension list all of it.
    # There an arrival that becomes the head of line drops the extension, and
    # the arrivals after it in the same batch follow requests that are no longer
    # listed: they must not be taken for the next ones.  300 replicas stop a few
    # requests around that length; then the others take arrivals again, and
    # migrations and admissions empty the queue in its order.
    R, I, S = 300, 65, 128
    cfg = _cfg(I, S, 600, dict(kind="poisson", mean=2.0), R=R, K=2, out=60.0)
    cfg["groups"][0]["tiers"] = dict(kind="explicit", probs=[0.05, 0.95])
    g, o = Scheduler(cfg), oracle.Oracle(cfg)
    g.queue_cache = ring
    g.set_queue_extension(64)

    def drain(flags):
        g.set_draining(flags)
        for r in range(R):
            for i in range(I):
                o.set_drain(r, i, bool(flags[r, i]))

    flags = np.ones((R, I), np.uint8)
    flags[:, 7] = 0
    drain(flags)
    g.step(ticks)
    o.step(ticks)
    waiting = ((g.export()["meta"].reshape(R, I, S)[:, 7] & 3) == 1).sum(1)
    assert waiting.min() < 66 + ring < waiting.max()
    drain(np.zeros((R, I), np.uint8))
    g.step(40)
    o.step(40)
    _same(g, o, "ring %d" % ring)
    assert g.stats()["raw"][86] == 0


BURSTS = dict(kind="gamma_poisson", mean=120.0, cv=3.0)
LONG_BURSTS = dict(kind="gamma_poisson", mean=300.0, cv=4.0)


@pytest.mark.parametrize("cfg,ring", [
    # piles longer than a full extension behind the ring: appends that end
    # there, insertions in front that push its last entry out
    (_cfg(65, 256, 420, BURSTS), 1),
    (_cfg(65, 256, 420, BURSTS), 15),
    (_cfg(130, 1024, 900, BURSTS, out=120.0), 3),
    (_cfg(256, 2048, 1500, LONG_BURSTS, interval=2, out=200.0), 11),
    (_cfg(129, 512, 700, LONG_BURSTS, K=1), 3),
    (_cfg(96, 192, 500, LONG_BURSTS, tier_blind=1), 7),
    (_cfg(100, 256, 500, LONG_BURSTS, dispatch=INFAAS), 7),
    (with_extensions(_cfg(70, 320, 500, LONG_BURSTS)), 7),
], ids=["I65_ring1", "I65_ring15", "I130", "I256", "one_tier", "blind", "infaas", "ext"])
@pytest.mark.parametrize("depth", [64, 100])
def test_a_full_extension_never_changes_a_result(cfg, ring, depth):
    g, o = Scheduler(cfg), oracle.Oracle(cfg)
    g.queue_cache = ring
    g.set_queue_extension(depth)
    longest = 0
    for ticks in (40, 40, 39, 41):
        g.step(ticks)
        o.step(ticks)
        _same(g, o, "tick %d" % g.tick)
        st = g.export()["meta"].reshape(-1, cfg["slots_per_instance"])
        longest = max(longest, int(((st & 3) == 1).sum(1).max()))
    assert g.stats()["raw"][86] == 0
    # some queue was longer than head, ring and extension, and requests entered
    # queues in the middle: preempted ones, or moved ones
    raw = o.export()["stats"].reshape(2, -1).sum(0)
    assert longest > 1 + ring + depth
    assert raw[5:80:8].sum() > 0 and ("dispatch" in cfg or raw[80] > 0)
