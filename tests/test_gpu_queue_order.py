"""The order kept behind each head of line (the LDS queue cache and, for more
than 64 instances, its extension in the state buffer) under everything that
enters a queue: runs of arrivals on empty and on non-empty queues, preempted
and migrated requests that fall inside the kept order, rings that overflow.
Bit-exact against the oracle; the kept order is a performance structure and
must never change a result."""
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


def _cfg(I, S, M, arrival, K=10, blind=0, interval=1, out=40.0, infaas=False):
    c = preset("tiny")
    c.update(n_instances=I, slots_per_instance=S, kv_blocks=M, headroom_base=M / 8.0, headroom_decay=0.7, mig_interval=interval,
             mig_max_pairs=I // 2, mig_stage_blocks=4, arrival=arrival, prompt=dict(kind="uniform_int", lo=16, hi=600),
             output=dict(kind="geometric", mean=out), groups=[dict(n_replicas=2, K=K, tiers=dict(kind="uniform"))], seed=77)
    if blind:
        c["tier_blind"] = 1
    if infaas:
        c["dispatch"] = dict(INFAAS)
    return c


POISSON = dict(kind="poisson", mean=14.0)
BURSTS = dict(kind="gamma_poisson", mean=30.0, cv=3.0)
WIDE_BURSTS = dict(kind="gamma_poisson", mean=120.0, cv=3.0)


@pytest.mark.parametrize("cfg,depths", [
    # short queues on few instances; the ring fills, overflows and drains
    (_cfg(3, 128, 500, POISSON), (0, 1, 2, 7, 15)),
    (_cfg(17, 64, 260, BURSTS), (1, 3, 7)),
    (_cfg(33, 192, 400, BURSTS, K=3), (0, 3, 7)),
    (_cfg(64, 64, 300, dict(kind="gamma_poisson", mean=60.0, cv=2.0)), (3, 7)),
    # one tier or tier-blind: every arrival follows the kept order
    (_cfg(5, 192, 400, BURSTS, K=1), (1, 7)),
    (_cfg(16, 128, 300, BURSTS, blind=1), (3, 7)),
    (_cfg(16, 128, 300, POISSON, infaas=True), (1, 7)),
    # INFaaS rounds: bursts of several batches, instances that fill up
    (_cfg(5, 64, 300, BURSTS, infaas=True), (0, 7)),
    (_cfg(64, 64, 200, dict(kind="gamma_poisson", mean=90.0, cv=2.0), infaas=True), (0, 3)),
    # the eight-wave kernels: piles beyond the ring go on in the extension,
    # preempted and migrated requests enter it in the middle
    (_cfg(65, 256, 420, WIDE_BURSTS), (1, 7, 15)),
    (_cfg(130, 1024, 900, WIDE_BURSTS, out=120.0), (0, 3, 11)),
    (_cfg(256, 2048, 1500, dict(kind="gamma_poisson", mean=300.0, cv=4.0), interval=2, out=200.0), (3, 11)),
])
def test_kept_queue_order_never_changes_a_result(cfg, depths):
    ticks = 160
    o = oracle.Oracle(cfg)
    o.step(ticks)
    want = o.export()
    for depth in depths:
        g = Scheduler(cfg)
        g.queue_cache = depth
        g.step(ticks - 41)
        g.step(41)
        got = g.export()
        for k in want:
            assert np.array_equal(got[k], want[k]), "I=%d depth %d field %s" % (cfg["n_instances"], depth, k)
        assert g.stats()["raw"][86] == 0
    # the workload reaches what it is there for: preempted and (under Llumnix)
    # moved requests enter the queues
    raw = want["stats"].reshape(2, -1).sum(0)
    assert raw[5:80:8].sum() > 0 and ("dispatch" in cfg or raw[80] > 0)


def test_depth_is_kept_where_every_replica_stays_resident():
    # 960 replicas of 32 instances: a cache fits beside them all
    cfg = preset("sweep")
    for grp in cfg["groups"]:
        grp["n_replicas"] = 32
    g = Scheduler(cfg)
    assert g.queue_cache > 0


@pytest.mark.parametrize("cfg,chosen", [
    (_cfg(16, 128, 300, dict(kind="poisson", mean=9.0)), 64),
    (_cfg(33, 192, 300, dict(kind="gamma_poisson", mean=20.0, cv=2.0), K=4, interval=3), 256),
    (_cfg(64, 64, 160, dict(kind="poisson", mean=24.0), blind=1), 256),
    (_cfg(17, 64, 200, dict(kind="poisson", mean=9.0), infaas=True), 64),
    (with_extensions(_cfg(20, 128, 200, dict(kind="poisson", mean=9.0))), 256),
], ids=["I16", "I33", "I64_blind", "I17_infaas", "I20_ext"])
def test_four_waves_per_replica_equal_one(cfg, chosen):
    # overloaded clusters can run four waves per replica or one (256 or 64
    # threads), and run four where they are expected to preempt often
    o = oracle.Oracle(cfg)
    o.step(200)
    want = o.export()
    assert want["stats"].reshape(2, -1)[:, :80].reshape(2, 10, 8)[:, :, 5].sum() > 0  # preemptions
    for threads in (0, 64, 256):
        g = Scheduler(cfg)
        g.set_launch(threads, 0)
        assert g.launch()[0] == (threads or chosen)
        g.step(150)
        g.set_launch(0, 1)  # back to the automatic size, both replicas in one block
        assert g.launch()[0] == chosen
        g.step(50)
        got = g.export()
        for k in want:
            assert np.array_equal(got[k], want[k]), "%d threads, field %s" % (threads, k)
    g.queue_cache = 0  # the four-wave kernels need a queue cache
    assert g.launch()[0] == 64
    with pytest.raises(MtsError):
        g.set_launch(128, 0)


@pytest.mark.parametrize("name,I,mean,kw,threads", [
    # overloaded, but long requests grow slowly and few are preempted: four
    # waves are slower (1024 replicas, 100 ticks: 1.90 ms against 1.75)
    ("gauss10", 16, 5.2, {}, 64),
    ("gauss10", 32, 10.4, {}, 64),
    ("gauss10", 56, 18.2, {}, 256),
    ("gauss10", 48, 15.6, dict(dispatch=INFAAS), 64),
    ("gauss10", 64, 20.8, dict(dispatch=INFAAS), 256),
    ("enterprise", 16, 11.4, {}, 256),
    ("sweep", 32, 30.0, {}, 256),
    # promotion passes bring rescans
    ("gauss10", 16, 5.2, dict(ext=True), 256),
])
def test_four_waves_where_a_cluster_preempts_often(name, I, mean, kw, threads):
    c = preset(name)
    c.update(n_instances=I, mig_max_pairs=I // 2, arrival=dict(kind="poisson", mean=mean))
    if kw.get("ext"):
        c = with_extensions(c)
    else:
        c.update(kw)
    c["groups"] = [dict(c["groups"][-1], n_replicas=8)]
    assert Scheduler(c).launch()[0] == threads


def test_one_wave_where_the_load_leaves_no_queue():
    assert Scheduler(preset("enterprise")).launch()[0] == 64
    g = Scheduler(preset("tiny"))
    assert g.launch()[0] == 64
    with pytest.raises(MtsError):
        g.set_launch(256, 0)


@pytest.mark.parametrize("cfg,depth", [
    # runs that end inside a word of slots, fill instances one after the other,
    # are more than the list of deferred runs holds, or fill the cluster
    (_cfg(65, 128, 300, dict(kind="gamma_poisson", mean=400.0, cv=3.0), out=20.0), 0),
    (_cfg(65, 128, 300, dict(kind="gamma_poisson", mean=400.0, cv=3.0), out=20.0), 7),
    (_cfg(129, 512, 700, dict(kind="gamma_poisson", mean=300.0, cv=4.0), K=1), 3),
    (_cfg(96, 192, 500, dict(kind="gamma_poisson", mean=300.0, cv=3.0), blind=1), 7),
    (_cfg(100, 256, 500, dict(kind="gamma_poisson", mean=200.0, cv=4.0), infaas=True), 7),
    (with_extensions(_cfg(70, 320, 500, dict(kind="gamma_poisson", mean=200.0, cv=4.0))), 7),
], ids=["depth0", "fills", "one_tier", "blind", "infaas", "ext"])
def test_long_bursts_placed_by_all_waves(cfg, depth):
    g, orc = Scheduler(cfg), oracle.Oracle(cfg)
    g.queue_cache = depth
    flags = np.zeros(2 * cfg["n_instances"], np.uint8)
    for ticks, drained in ((40, ()), (50, (0, 5, 64)), (50, (0, 64))):
        for i in range(cfg["n_instances"]):
            orc.set_drain(0, i, i in drained)
            flags[i] = i in drained
        g.set_draining(flags)
        g.step(ticks)
        orc.step(ticks)
        got, want = g.export(), orc.export()
        for k in want:
            assert np.array_equal(got[k], want[k]), "depth %d field %s" % (depth, k)
        assert g.stats()["raw"][86] == 0
