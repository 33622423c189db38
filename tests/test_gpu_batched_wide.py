"""Continuous batching on pools beyond one segment of lanes: the multi-wave
kernel at the edges of its classes (129 instances up, pools that leave waves
without instances, the widest), every policy and backlog, ties, more
departures at once than a wave lists, a full ring; and the pools that still
take the general kernel."""
import numpy as np
import pytest
import torch

from paper_2609_16206_amd import rt_router as R
from paper_2609_16206_amd import workload as W
from tests.gpu_common import log, run_sim
from tests.parity import check_properties, follow_replicas, goodput_recount

pytestmark = pytest.mark.gpu

MODES = [("learned", "true"), ("learned", "proxy"), ("round_robin", "true"), ("least_loaded", "true"),
         ("learned_sampled", "true"), ("learned_sampled", "proxy"), ("length_threshold", "true")]


def _points(P, D, **kw):
    return [dict(W.make_point(P, D, n_classes=3, policy=pol, backlog_mode=bm, kv_cap=20_000, len_threshold=150,
                              service="batched", **kw), batch_cap=1024) for pol, bm in MODES]


def _trace(pts, lens, rate, seed=51):
    traf = W.mixed_bursty()
    traf = traf.scaled(rate * W.capacity_rps(pts[0], traf) / traf.mean_rate())
    parts = [W.replica_arrays(seed, i, traf, n) for i, n in enumerate(lens)]
    tr = {k: np.concatenate([q[k] for q in parts]) for k in parts[0]}
    tr["offsets"] = np.concatenate(([0], np.cumsum(lens))).astype(np.int64)
    tr["param_point"] = (np.arange(len(lens)) % len(pts)).astype(np.int32)
    W.add_sample_words(tr, seed)
    return tr


def _check(pts, tr, what):
    gpu, g, met, flags = run_sim(pts, tr)
    assert flags & ~1 == 0
    check_properties(pts, tr, gpu)
    assert np.array_equal(goodput_recount(pts, tr, gpu), met)
    rep = follow_replicas(pts, tr, gpu, range(len(tr["offsets"]) - 1), gpu_goodput=g, gpu_met=met)
    log(f"batched {what}: {rep}")
    return flags


@pytest.mark.parametrize("P,D", [(64, 65), (1, 130), (130, 1), (3, 252), (5, 252), (2, 500), (200, 220), (300, 600),
                                 (128, 1024), (1024, 300), (900, 900)])
def test_pools_beyond_a_segment(P, D):
    pts = _points(P, D)
    assert _check(pts, _trace(pts, [181, 64, 1, 200, 150, 0, 333, 97, 120, 2, 250, 77, 130, 300], 2.0), f"{P}+{D}") == 0


def test_ties_and_rejections():
    pts = _points(20, 120, beta_pre=1.0, beta_dec=0.25)
    tr = _trace(pts, [400] * 14, 4.0)
    tr["arrival_ns"] = tr["arrival_ns"] // 50_000_000 * 50_000_000
    bad = np.random.default_rng(1).choice(tr["arrival_ns"].size, 40, replace=False)
    tr["prompt_len"][bad[::2]] = 0
    tr["slo_class"][bad[1::2]] = 3
    assert _check(pts, tr, "ties and rejections") == 1


def test_more_departures_than_a_list():
    """3,000 requests at one time on 1,024 prefill instances, then one much
    later: every wave has several rounds of 128 departures to hand over."""
    pts = _points(1024, 200)[:1]
    tr = _trace(pts, [3002], 1.0)
    tr["arrival_ns"][:] = 1000
    tr["arrival_ns"][-1] = 10 ** 12
    assert _check(pts, tr, "departures") == 0


def test_full_ring_stops_the_replica():
    pts = [dict(p, batch_cap=2) for p in _points(4, 140)[:1]]
    tr = _trace(pts, [300, 3], 8.0)
    tr["arrival_ns"][:300] //= 64
    _, _, _, flags = run_sim(pts, tr)
    assert flags == 8


def test_scratch_is_one_pool_of_rings_a_replica():
    """32 bytes a ring place, P + D instances a replica: 604 MB for one replica of 32 + 256 with the largest batch_cap,
    and no more than that is taken."""
    pt = dict(W.make_point(32, 256, n_classes=3, service="batched"), batch_cap=65536)
    tr = _trace([pt], [300], 2.0)
    sim = R.Simulator([pt])
    dtr = R.to_device(tr)
    out = R.alloc_outputs(300)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    sim.run(dtr, out)
    torch.cuda.synchronize()
    taken = before - torch.cuda.mem_get_info()[0]
    flags = sim.data_status()
    sim.close()
    assert flags == 0 and taken <= 288 * 65536 * 32 + (64 << 20), taken
    gpu = {k: v.cpu().numpy() for k, v in out.items()}
    follow_replicas([pt], tr, gpu, [0])
