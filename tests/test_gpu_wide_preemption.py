"""Preemption in the kernels for more than 64 instances: up to four preempting
instances of a tick are scanned by all waves together, more of them one by
each wave.  Bit-exact against the oracle where calls take several victims."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from workloads import preset, with_extensions  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU-only hosts, never run there
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2608_16336_amd import Scheduler  # noqa: E402


def _cfg(I, S, M, mean, hi=40, out=60.0, block=16, blind=0, infaas=False):
    c = preset("tiny")
    c.update(n_instances=I, slots_per_instance=S, kv_blocks=M, block_tokens=block, headroom_base=M / 16.0, headroom_decay=0.6,
             mig_interval=1, mig_max_pairs=I // 2, mig_stage_blocks=2, arrival=dict(kind="gamma_poisson", mean=mean, cv=2.0),
             prompt=dict(kind="uniform_int", lo=8, hi=hi), output=dict(kind="geometric", mean=out),
             groups=[dict(n_replicas=2, K=10, tiers=dict(kind="uniform"))], seed=9)
    if blind:
        c["tier_blind"] = 1
    if infaas:
        c["dispatch"] = dict(policy="infaas", alpha=64, beta=1, gamma=1, pen_overloaded=512, pen_interfered=128, ewma_shift=4)
    return c


CASES = dict(
    # small requests: a victim frees a block or two, a tick's growth takes several
    few=_cfg(65, 64, 40, 14.0),
    many=_cfg(70, 128, 60, 60.0),
    every_chunk=_cfg(80, 2048, 400, 400.0, hi=20, out=120.0, block=8),
    odd_chunks=_cfg(129, 704, 300, 200.0, hi=600),
    blind=_cfg(96, 192, 80, 60.0, blind=1),
    infaas=_cfg(100, 256, 60, 60.0, infaas=True),
    ext=with_extensions(_cfg(72, 320, 60, 50.0)),
)


@pytest.mark.parametrize("name", list(CASES))
def test_preemption_by_all_waves(name):
    cfg = CASES[name]
    o = oracle.Oracle(cfg)
    o.step(120)
    want = o.export()
    assert want["stats"].reshape(2, -1)[:, :80].reshape(2, 10, 8)[:, :, 5].sum() > 100  # preemptions
    for depth in (0, 7):
        g = Scheduler(cfg)
        g.queue_cache = depth
        g.step(77)
        g.step(43)
        got = g.export()
        for k in want:
            assert np.array_equal(got[k], want[k]), "%s depth %d field %s" % (name, depth, k)
        assert g.stats()["raw"][86] == 0
