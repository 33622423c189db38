"""The one-wave kernel with its FIFOs in LDS (pools of at most 32 instances a
side) where its ring can go wrong: queues far beyond the ring that then drain
many requests between two arrivals (refills one step ahead and at once), the
edges of the segment widths, every scoring mode, few replicas (large rings)
and many (small ones); and launches of several threads."""
import threading

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


@pytest.mark.parametrize("n_rep,n_req", [(14, 3001), (3584, 130)])
@pytest.mark.parametrize("P,D", [(1, 1), (4, 4), (5, 3), (8, 8), (2, 9), (16, 16), (17, 1), (32, 32)])
def test_deep_rings_that_drain(P, D, n_rep, n_req):
    pts = [W.make_point(P, D, n_classes=3, policy=pol, backlog_mode=bm, kv_cap=20_000, len_threshold=150)
           for pol, bm in MODES]
    traf = W.mixed_bursty()
    # bursts of 60 to 700 requests at six times the capacity, then a lull that
    # lets about two thirds of the queue finish before the next arrival
    k = 6.0 * W.capacity_rps(pts[0], traf) / traf.mean_rate()
    rng = np.random.default_rng(P * 64 + D)
    lens = n_req - np.arange(n_rep) % 5
    parts = []
    for i in range(n_rep):
        d = W.replica_arrays(43, i, traf.scaled(k), int(lens[i]))
        gaps = np.diff(d["arrival_ns"], prepend=0)
        at = np.cumsum(rng.integers(60, 700, 64))
        at = at[at < lens[i]]
        gaps[at] += (0.66 * np.diff(d["arrival_ns"][at], prepend=0) * 5.0).astype(np.int64)
        d["arrival_ns"] = np.cumsum(gaps)
        parts.append(d)
    tr = {key: np.concatenate([q[key] for q in parts]) for key in parts[0]}
    tr["offsets"] = np.concatenate(([0], np.cumsum(lens))).astype(np.int64)
    tr["param_point"] = (np.arange(n_rep) % len(pts)).astype(np.int32)
    W.add_sample_words(tr, 9)
    gpu, g, met, flags = run_sim(pts, tr)
    assert flags == 0
    check_properties(pts, tr, gpu)
    assert np.array_equal(goodput_recount(pts, tr, gpu), met)
    reps = range(n_rep) if n_rep < 100 else range(0, n_rep, 31)
    rep = follow_replicas(pts, tr, gpu, reps, gpu_goodput=g, gpu_met=met)
    log(f"LDS FIFOs {P}+{D}, {n_rep} x {n_req}: {rep}")


# Launch sizes on both sides of each line at which a pool changes its kernel, its ring length or the workgroups that
# share a compute unit: a ragged last workgroup, 5 to 7, 9 to 12 and 13 to 16 waves a compute unit, segments of four
# lanes.
@pytest.mark.parametrize("P,D,n_rep", [(2, 6, 4610), (2, 6, 9001), (2, 6, 13001), (2, 6, 17003), (3, 3, 9002), (4, 1, 6200),
                                       (8, 1, 4107), (9, 1, 1601), (8, 8, 5003), (8, 8, 9005), (5, 5, 9001), (8, 2, 33001),
                                       (2, 12, 33001), (16, 16, 3001), (24, 3, 1030), (32, 32, 601), (2, 32, 1501)])
def test_launch_sizes(P, D, n_rep):
    pts = [W.make_point(P, D, n_classes=3, policy=pol, backlog_mode=bm, kv_cap=20_000, len_threshold=150)
           for pol, bm in MODES]
    # (one mode a call, so that the call has the launch size of that mode's class; every replica one of 32 traces)
    traf = W.mixed_bursty()
    traf = traf.scaled(1.2 * W.capacity_rps(pts[0], traf) / traf.mean_rate())
    parts = [W.replica_arrays(61, i, traf, 70 - i % 5) for i in range(32)]
    for pt in pts:
        rep = [parts[i % 32] for i in range(n_rep)]
        tr = {key: np.concatenate([q[key] for q in rep]) for key in parts[0]}
        lens = [70 - (i % 32) % 5 for i in range(n_rep)]
        tr["offsets"] = np.concatenate(([0], np.cumsum(lens))).astype(np.int64)
        tr["param_point"] = np.zeros(n_rep, np.int32)
        if pt["policy"] == "learned_sampled":
            W.add_sample_words(tr, 11)
        gpu, g, met, flags = run_sim([pt], tr)
        assert flags == 0
        check_properties([pt], tr, gpu)
        follow_replicas([pt], tr, gpu, range(0, n_rep, n_rep // 60), gpu_goodput=g, gpu_met=met)
        if pt["policy"] != "learned_sampled":  # replicas of one trace are alike, in whichever wave
            k = sum(lens[:32])
            for key in gpu:
                whole = gpu[key][: len(gpu[key]) // k * k].reshape(-1, k)
                assert (whole == whole[0]).all(), key


@pytest.mark.parametrize("service,P,D", [("serial", 16, 16), ("batched", 40, 80)])
def test_launches_of_two_threads_with_unequal_rings(service, P, D):
    """Two host threads, each with a simulator and a stream of its own, launch the same kernel class with different
    amounts of LDS: neither refuses the other's launch, and every call gives the first one's outputs."""
    pt = W.make_point(P, D, n_classes=3, service=service)
    failed = []

    def work(n_rep):
        try:
            tr = R.to_device(W.make_trace(W.Workload("threads", 3, n_rep, 40, [pt], [W.mixed_bursty()])))
            sim = R.Simulator([pt])
            stream = torch.cuda.Stream()
            first = None
            for _ in range(60):
                with torch.cuda.stream(stream):
                    out = sim.run(tr, stream=stream)
                stream.synchronize()
                got = {k: v.cpu() for k, v in out.items()}
                first = first or got
                assert all(torch.equal(first[k], got[k]) for k in got)
            sim.close()
        except Exception as e:  # (an assertion in a thread is not the test's own)
            failed.append(e)

    threads = [threading.Thread(target=work, args=(n,)) for n in (3, 300)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
