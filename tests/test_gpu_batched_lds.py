"""Continuous batching in one wave: queues that outgrow their rings in LDS
(sorted on into HBM and back), departures at once beyond a segment's list, a
prefill so long that its decode placement is read back from the output, and
launches of so many waves that a ring is a few entries; joins and completions
at one instant, and requests without prefill work next to replicas whose lists
are full; and rejections around the request that finds a queue full."""
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


# Traces on a grid of 1 ns (beta, first arrival, arrivals after it, prompts; one ns a token) in which a request
# arrives just where a member's completion, taken again from the clock at that arrival, rounds to.  The request is
# in the batch by then; were the member to leave first, a TTFT would differ by 1 ns.
ROUNDED_TO_ARRIVAL = [
    (0.25, 23925, [0, 0, 3, 7, 7, 11], [5, 3, 6, 4, 2, 2]),
    (0.25, 16992, [0, 4, 7, 11, 12], [7, 5, 4, 3, 2]),
    (0.25, 1863, [0, 3, 6, 6, 9, 13, 14, 18, 19], [2, 3, 4, 4, 4, 6, 2, 7, 5]),
    (0.25, 24298, [0, 4, 7, 8, 11, 14, 15, 19, 23, 27, 27], [3, 3, 5, 4, 3, 5, 5, 5, 5, 4, 7]),
    (0.5, 25912, [0, 0, 0, 2, 2, 5, 9, 10, 12], [1, 5, 3, 2, 5, 2, 4, 6, 2]),
    (0.5, 25319, [0, 2, 2, 4, 7, 11, 12], [5, 7, 3, 7, 2, 5, 1]),
]


def _fine_points(shapes, betas):
    return [dict(W.make_point(P, D, n_classes=1, policy="round_robin", service="batched"), batch_cap=1024, beta_pre=b,
                 beta_dec=b, pre_base_ns=0, pre_tok_ns=1, dec_tok_ns=1, xfer_tok_ns=1) for P, D in shapes for b in betas]


def _fine_trace(replicas, point_of):
    """Replicas of (arrivals, prompts, outputs) as one trace."""
    lens = [len(a) for a, _, _ in replicas]
    tr = dict(arrival_ns=np.concatenate([a for a, _, _ in replicas]).astype(np.int64),
              prompt_len=np.concatenate([p for _, p, _ in replicas]).astype(np.int32),
              out_len=np.concatenate([o for _, _, o in replicas]).astype(np.int32))
    tr["pred_out_len"] = tr["out_len"].copy()
    tr["slo_class"] = np.zeros(len(tr["out_len"]), np.uint8)
    tr["offsets"] = np.concatenate(([0], np.cumsum(lens))).astype(np.int64)
    tr["param_point"] = np.asarray(point_of, np.int32)
    return tr


# Every segment width (so many replicas that the launch keeps it narrow), two instances a lane, one replica a workgroup.
@pytest.mark.parametrize("D,n", [(1, 8400), (6, 4200), (14, 2100), (30, 1056), (60, 6), (126, 6), (140, 6)])
def test_join_before_a_completion_that_rounds_to_its_arrival(D, n):
    pts = _fine_points([(1, D)], [0.25, 0.5])
    reps = [(t0 + np.array(a), p, np.ones(len(a))) for _, t0, a, p in ROUNDED_TO_ARRIVAL]
    point_of = [0 if b == 0.25 else 1 for b, *_ in ROUNDED_TO_ARRIVAL]
    tr = _fine_trace(reps * (n // 6), point_of * (n // 6))
    assert _check(pts, tr, f"rounded to an arrival, 1+{D}") == 0


def test_short_traces_on_a_fine_grid():
    pts = _fine_points([(1, 1), (2, 2), (1, 6), (3, 1)], [0.25, 0.5, 1.0, 1.0 / 3.0])
    rng = np.random.default_rng(17)
    reps = []
    for i in range(4000):
        n = int(rng.integers(4, 32))
        reps.append((rng.integers(0, 30_000) + np.cumsum(rng.integers(0, 5, n)), rng.integers(1, 8, n), rng.integers(1, 8, n)))
    assert _check(pts, _fine_trace(reps, np.arange(4000) % len(pts)), "fine grid") == 0


@pytest.mark.parametrize("P,D,n_rep", [(5, 3, 4200), (9, 7, 2100), (20, 11, 1060), (40, 23, 20), (90, 37, 20)])
def test_no_prefill_work_beside_full_lists(P, D, n_rep):
    """Replicas whose prefill instances all end a request at one time, more at once than a segment lists, in waves
    with replicas whose requests take no time to prefill."""
    base = W.make_point(P, D, n_classes=1, policy="round_robin", service="batched", beta_pre=0.0)
    pts = [dict(base, batch_cap=1024), dict(base, batch_cap=1024, pre_base_ns=0, pre_tok_ns=0, xfer_tok_ns=0)]
    n = 6 * P + 3
    burst = np.arange(n) // P * 10**10
    reps = [(burst, np.full(n, 100), np.full(n, 20)), (np.arange(n) * 7_000_000, np.full(n, 100), np.full(n, 20))]
    tr = _fine_trace(reps * (n_rep // 2), np.arange(n_rep) % 2)
    assert _check(pts, tr, f"no prefill work {P}+{D}") == 0


@pytest.mark.parametrize("late", [False, True])
@pytest.mark.parametrize("where", ["prefill", "transfers", "decode"])
@pytest.mark.parametrize("width", [1, 40, 100, 200, 1024])  # the instances on the side that does not overflow
def test_rejections_around_a_full_queue(width, where, late):
    """A replica stops at the request that finds a queue full: requests after it are not looked at, so a bad one
    among them sets no flag; one before it does."""
    P, D = (1, width) if where == "prefill" else (width, 1)
    pt = dict(W.make_point(P, D, n_classes=1, policy="round_robin", service="batched"), batch_cap=2)
    n = 8
    gap = 0 if where == "prefill" else 10**12
    if where == "transfers":
        pt.update(xfer_tok_ns=1 << 40)
    elif where == "decode":
        pt.update(xfer_tok_ns=0, dec_tok_ns=1 << 40)
    # the third request (transfer, decode member) is one too many: found at its own admission, or by the arrival after
    stop = 2 if where == "prefill" else 3
    bad = stop + 1 if late else stop - 1
    tr = _fine_trace([(np.arange(n) * gap, np.full(n, 100), np.full(n, 20))], [0])
    tr["prompt_len"][bad] = 0
    flags = run_sim([pt], tr)[3]
    assert flags & ~4 == (8 if late else 9)


# 5 to 7 and 9 to 11 waves a compute unit (and a ragged last workgroup).
@pytest.mark.parametrize("P,D,n", [(2, 6, 4610), (2, 6, 8300), (1, 2, 17100), (3, 14, 2500), (3, 14, 4200), (12, 20, 4600),
                                   (10, 29, 1300), (10, 29, 2070), (1, 31, 4300), (2, 62, 2300), (32, 32, 3080),
                                   (8, 64, 1100)])
def test_waves_between_whole_workgroups(P, D, n):
    # with and without candidate words, which take room from the rings
    for pts in (_points(P, D), _points(P, D)[:4]):
        tr = _bursts(pts, [20 - (i % 5) for i in range(n)], 10, 10**9)
        if len(pts) == 4:
            del tr["sample_bits"]
        gpu, g, met, flags = run_sim(pts, tr)
        assert flags == 0
        check_properties(pts, tr, gpu)
        follow_replicas(pts, tr, gpu, range(0, n, n // 60), gpu_goodput=g, gpu_met=met)
