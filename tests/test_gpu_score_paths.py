"""The standalone scorer's branches: the shared-snapshot loop that takes costs
four at a time (and what must keep out of it), and the lanes-per-request
kernel over widths around its lane counts, with one snapshot and with rows."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2609_16206_amd import workload as W
from tests.test_gpu_score import _compare, _gpu_score

pytestmark = pytest.mark.gpu


def _spoil(kind, d, prm):
    """Values that the four-at-a-time loop does not take, and some it does."""
    w = d["queue"].size
    if kind == "rho 2.5":
        prm["rho"] = 2.5
    elif kind == "zero weights":  # every cost 0: the lowest index wins
        prm.update(w_b=-0.0, w_s=0.0, w_q=-0.0)
    elif kind == "equal":
        for k in ("queue", "kv_occ", "backlog_s"):
            d[k][:] = d[k][0]
    elif kind == "occupancy 2^24":
        d["kv_occ"][w // 2] = (1 << 24) - 300  # + need: above 2^24 for most requests
    elif kind == "occupancy 2^31":
        d["kv_occ"][::2] = (1 << 31) - 1  # + need: above 2^31
    elif kind == "negative occupancy":
        d["kv_occ"][w - 1] = -70_000
    elif kind == "infinite cost":
        prm["w_b"] = 3e38  # w_b * backlog beyond float32: +inf
        d["backlog_s"][: max(1, w // 2)] = 9.0
    elif kind == "nan cost":
        prm.update(w_s=3e38, rho=3e38, sigma=[0.0, 2.0] + [1.0] * 6)  # inf * 0


@pytest.mark.parametrize("kind", ["plain", "rho 2.5", "zero weights", "equal", "occupancy 2^24", "occupancy 2^31",
                                  "negative occupancy", "infinite cost", "nan cost"])
@pytest.mark.parametrize("n_inst", [1, 3, 4, 5, 9, 10, 11, 12, 13, 64, 67])
def test_shared_snapshot_loops(n_inst, kind):
    d = W.scorer_inputs(n_req=(1 << 16) + 3, n_inst=n_inst, seed=20 + n_inst)
    prm = W.scorer_params()
    _spoil(kind, d, prm)
    d["prompt_len"][5::1009] = 0
    for pool in ("decode", "prefill"):
        if kind != "nan cost":
            _compare(prm, pool, d, n_inst, 0, d["kv_cap"])
            continue
        # (the sign of a NaN is the host's or the GPU's own)
        gi, gs = _gpu_score(prm, pool, d, d["prompt_len"].size, n_inst, 0, d["kv_cap"])
        oi, os_, _ = O.score(prm, pool, d["backlog_s"], d["queue"], d["kv_occ"], d["kv_cap"], n_inst, 0, d["prompt_len"],
                             d["pred_out_len"], d["slo_class"])
        assert np.isnan(os_[oi >= 0]).any()
        np.testing.assert_array_equal(gi, oi)
        np.testing.assert_array_equal(gs, os_)


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n_inst,stride", [(1, 1), (1, 3), (2, 2), (2, 5), (3, 3), (5, 7), (15, 15), (16, 17), (17, 17), (33, 35), (48, 49), (63, 63),
                                           (64, 65), (127, 127), (128, 131), (193, 193), (257, 259)])
def test_lanes_per_request(n_inst, stride, shared):
    n_req = 1031
    w = n_inst if shared else stride
    d = W.scorer_inputs(n_req=n_req, n_inst=w, seed=300 + n_inst, per_request=not shared)
    d["prompt_len"][3::101] = 0
    d["kv_occ"][w - 1] = -1234
    prm = W.scorer_params()
    _compare(prm, "decode", d, n_inst, 0 if shared else stride, d["kv_cap"])
    _compare(prm, "prefill", d, n_inst, 0 if shared else stride, d["kv_cap"])
