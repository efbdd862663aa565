"""Step launches take up the summaries that the last launch left; whatever
changes the state, the clock or the layout in between makes them start from
the slots again.  Bit-exact against the oracle through every such call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import scaled, with_extensions  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU-only hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_16336_amd import Scheduler  # noqa: E402
from paper_2608_16336_amd.mts import MtsError  # noqa: E402

INFAAS = dict(policy="infaas", alpha=64, beta=1, gamma=1, pen_overloaded=512, pen_interfered=128, ewma_shift=4)


def _cfg(name, **kw):
    c = scaled(name, replicas_per_group=3)
    c["groups"] = [dict(c["groups"][0], n_replicas=3)]
    c["arrival"]["mean"] *= kw.pop("load", 1.0)
    if kw.pop("ext", False):
        c = with_extensions(c)
    c.update(kw)
    return c


def _same(g, orc, what):
    for r, o in enumerate(orc):
        a, b = g.export(r, 1), o.export()
        for k in b:
            assert np.array_equal(a[k], b[k]), "%s: replica %d field %s" % (what, r, k)


@pytest.mark.parametrize("cfg", [
    _cfg("tiny", load=2.0), _cfg("enterprise", load=1.5), _cfg("gauss10", ext=True), _cfg("sweep", load=2.5),
    _cfg("enterprise", load=1.3, dispatch=INFAAS, tier_blind=1), _cfg("wide"), _cfg("wide", ext=True),
], ids=["tiny", "enterprise", "gauss10_ext", "sweep", "infaas_blind", "wide", "wide_ext"])
def test_launches_resume_through_every_change_of_state(cfg):
    g = Scheduler(cfg)
    orc = [oracle.Oracle(cfg, r, 1) for r in range(g.R)]
    I = cfg["n_instances"]

    def step(n, noalloc=False):
        (g.step_noalloc if noalloc else g.step)(n)
        for o in orc:
            o.step(n)

    step(60)
    step(1)
    step(7)
    _same(g, orc, "short steps")
    flags = np.zeros((g.R, I), np.uint8)
    flags[:, :max(1, I // 4)] = 1
    g.set_draining(flags)
    for o in orc:
        for i in range(max(1, I // 4)):
            o.set_drain(0, i, True)
    step(6)
    _same(g, orc, "draining")
    # one replica takes another's state, the others go on from their images
    saved = g.export(0, 1)
    g.import_state(saved, 1, 1)
    orc[1].import_state(saved)
    step(5)
    _same(g, orc, "one replica imported")
    depth = g.queue_cache
    g.queue_cache = 1
    step(4)
    g.queue_cache = depth
    step(3)
    _same(g, orc, "queue cache depth changed")
    g.set_wheel_cap(max(1, g.wheel()[1] // 8))
    step(9)
    _same(g, orc, "wheel capacity changed")
    t = g.tick
    g.tick = t + 1000
    g.tick = t
    step(2)
    step(3, noalloc=True)
    step(2)
    _same(g, orc, "clock moved back and forth")
    # a launch that starts again at an earlier tick's state
    saved = [g.export(r, 1) for r in range(g.R)]
    step(8)
    for r in range(g.R):
        g.import_state(saved[r], r, 1)
        orc[r].import_state(saved[r])
    g.tick = t + 7
    for o in orc:
        o.tick = t + 7
    step(8)
    _same(g, orc, "rewound")
    assert g.stats()["raw"][86] == 0


@pytest.mark.parametrize("I,S", [(4, 64), (61, 576), (61, 1088), (201, 2048)])
def test_checkpoint_larger_than_one_slice_of_the_staging(I, S):
    # few sampled arrivals leave a staging area smaller than the slots, so the
    # canonical arrays of the largest state pass in four slices, the last one
    # partial; the smallest is converted by the host
    c = _cfg("tiny", n_instances=I, slots_per_instance=S, mig_max_pairs=I // 2)
    c["arrival"]["mean"] = 0.05
    c["groups"] = [dict(c["groups"][0], n_replicas=2)]
    g = Scheduler(c)
    orc = [oracle.Oracle(c, r, 1) for r in range(2)]
    rng = np.random.RandomState(5)
    st = g.export()
    N = I * S
    # requests all over the slots (waiting, lengths and tiers at random)
    for r in range(2):
        at = rng.choice(N, min(N // 2, 3000), replace=False) + r * N
        at[-1] = (r + 1) * N - 1
        at = np.unique(at)
        st["meta"][at] = 1 | (rng.randint(0, 2, len(at)) << 2)
        st["lr"][at] = rng.randint(1, 900, len(at)) | (rng.randint(1, 300, len(at)) << 16)
        st["seq"][at] = rng.permutation(len(at))
        st["next_seq"][r] = len(at)
    g.import_state(st)
    for k, v in g.export().items():
        assert np.array_equal(v, st[k]), k
    n = {k: len(v) // 2 for k, v in st.items()}
    for r, o in enumerate(orc):
        o.import_state({k: v[r * n[k]:(r + 1) * n[k]] for k, v in st.items()})
        o.step(20)
    g.step(20)
    _same(g, orc, "after the import")
    # a bad slot in the last slice refuses the whole state and changes nothing
    before = g.export()
    bad = {k: v.copy() for k, v in before.items()}
    bad["meta"][2 * N - 1] = 1 | (9 << 2)
    bad["seq"][0] ^= 1
    with pytest.raises(MtsError) as e:
        g.import_state(bad)
    assert e.value.code == -1
    for k, v in g.export().items():
        assert np.array_equal(v, before[k]), k
    g.step(5)
    for o in orc:
        o.step(5)
    _same(g, orc, "after the refused import")


def test_replicas_beyond_the_images_budget_start_from_their_slots():
    # 80,000 replicas of wide clusters with few slots and short outputs, 32 GB:
    # their images would take 9.6 GB, more than the budget of 8 GiB, so the last
    # ones have none; the others' steps resume from theirs
    R = 80000
    c = _cfg("wide", n_instances=129, slots_per_instance=64, kv_blocks=40, block_tokens=64, headroom_base=5.0, mig_max_pairs=64,
             arrival=dict(kind="gamma_poisson", mean=30.0, cv=2.0), prompt=dict(kind="uniform_int", lo=64, hi=1600),
             output=dict(kind="geometric", mean=1.5), groups=[dict(n_replicas=R, K=4, tiers=dict(kind="uniform"))])
    g = Scheduler(c)
    assert g.nbytes < 48 << 30
    at = (0, 40000, 71000, 72000, 79998, R - 1)
    orc = [oracle.Oracle(c, r, 1) for r in at]
    for n in (3, 1, 5, 2):
        g.step(n)
        for o in orc:
            o.step(n)
        for r, o in zip(at, orc):
            a, b = g.export(r, 1), o.export()
            for k in b:
                assert np.array_equal(a[k], b[k]), "replica %d field %s" % (r, k)
    # replicas without an image take a state as well
    saved = g.export(0, 1)
    g.import_state(saved, R - 1, 1)
    orc[-1].import_state(saved)
    g.step(4)
    for r, o in zip(at, orc):
        o.step(4)
        a, b = g.export(r, 1), o.export()
        for k in b:
            assert np.array_equal(a[k], b[k]), "replica %d field %s after the import" % (r, k)
    assert g.stats()["raw"][86] == 0
    g.close()
    torch.cuda.empty_cache()


def test_a_cache_deeper_than_the_images_have_room_for():
    # up to 64 instances the images have room for a ring of 7
    cfg = _cfg("enterprise", load=1.5)
    g = Scheduler(cfg)
    orc = [oracle.Oracle(cfg, r, 1) for r in range(g.R)]
    for depth, n in ((7, 30), (15, 20), (15, 3), (7, 2), (7, 3), (15, 1), (7, 4)):
        g.queue_cache = depth
        g.step(n)
        for o in orc:
            o.step(n)
        _same(g, orc, "depth %d" % depth)
    assert g.stats()["raw"][86] == 0


@pytest.mark.parametrize("replicas", [1, 40])
def test_a_state_loaded_on_one_stream_is_stepped_on_another(replicas):
    # small states are converted by the host, larger ones on the device: both
    # loads are complete when the call returns, whatever stream steps next
    c = _cfg("enterprise", load=1.3)
    c["groups"][0]["n_replicas"] = replicas
    g, o = Scheduler(c), oracle.Oracle(c, 0, 1)
    g.step(30)
    o.step(30)
    saved = g.export()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for k in range(6):
        g.step(8, stream=streams[k % 3])
        g.import_state(saved)
        g.tick = 30
        g.step(4, stream=streams[(k + 1) % 3])
        torch.cuda.synchronize()
    o.step(4)
    a, b = g.export(0, 1), o.export()
    for f in b:
        assert np.array_equal(a[f], b[f]), f
