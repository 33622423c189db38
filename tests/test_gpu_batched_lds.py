"""Continuous batching in one wave: queues that outgrow their rings in LDS
(sorted on into HBM and back), departures at once beyond a segment's list, a
prefill so long that its decode placement is read back from the output, and
launches of so many waves that a ring is a few entries."""
import numpy as np
import pytest

from paper_2609_16206_amd import workload as W
from tests.gpu_common import run_sim
from tests.parity import check_properties, follow_replicas, goodput_recount
from tests.test_gpu_batched_wide import _check, _points

pytestmark = pytest.mark.gpu


def _bursts(pts, lens, per_burst, gap_ns, seed=77):
    """Requests in bursts of `per_burst` at one instant, `gap_ns` apart."""
    traf = W.mixed_bursty()
    parts = [W.replica_arrays(seed, i, traf, n) for i, n in enumerate(lens)]
    for q, n in zip(parts, lens):
        q["arrival_ns"] = (np.arange(n) // per_burst * gap_ns).astype(np.int64)
    tr = {k: np.concatenate([q[k] for q in parts]) for k in parts[0]}
    tr["offsets"] = np.concatenate(([0], np.cumsum(lens))).astype(np.int64)
    tr["param_point"] = (np.arange(len(lens)) % len(pts)).astype(np.int32)
    W.add_sample_words(tr, seed)
    return tr


@pytest.mark.parametrize("P,D", [(1, 1), (1, 3), (6, 2), (2, 6), (13, 3), (1, 31), (30, 2), (56, 8), (100, 28), (1, 127)])
def test_bursts_beyond_rings_and_lists(P, D):
    pts = _points(P, D)
    # one burst of everything, then bursts a long and a short gap apart
    lens = [150, 97, 31, 0, 1, 160, 3, 90]
    for per, gap in ((1 << 20, 1), (120, 10**12), (25, 20_000_000)):
        assert _check(pts, _bursts(pts, lens, per, gap), f"bursts {P}+{D}") == 0


@pytest.mark.parametrize("P,D,n", [(2, 6, 9000), (1, 2, 17000), (30, 40, 2100)])
def test_many_waves(P, D, n):
    pts = _points(P, D)
    lens = [30 - (i % 7) for i in range(n)]
    tr = _bursts(pts, lens, 15, 10**9)
    gpu, g, met, flags = run_sim(pts, tr)
    assert flags == 0
    check_properties(pts, tr, gpu)
    assert np.array_equal(goodput_recount(pts, tr, gpu), met)
    follow_replicas(pts, tr, gpu, range(0, n, n // 40), gpu_goodput=g, gpu_met=met)


@pytest.mark.parametrize("P,D,n", [(3, 14, 6200), (10, 29, 3100)])
def test_three_waves_per_simd(P, D, n):
    pts = _points(P, D)
    tr = _bursts(pts, [20 - (i % 5) for i in range(n)], 10, 10**9)
    gpu, g, met, flags = run_sim(pts, tr)
    assert flags == 0
    check_properties(pts, tr, gpu)
    follow_replicas(pts, tr, gpu, range(0, n, n // 40), gpu_goodput=g, gpu_met=met)
