"""Which controlled phases run together, as the work counts report it (host only)."""

import numpy as np
import pytest

from paper_2010_09746_amd import costmodel
from paper_2010_09746_amd import qsim as Q
from workloads import KIND_CU, KIND_U, haar_u2, make_gates, phase, qft_circuit


def _counts(g, n, k, **kw):
    p = Q.Program(g, n, "c128", **{**dict(form="pass", k_tile=k, max_swaps=4, pinned=3, perm_exec="relabel"), **kw})
    c = p.op_counts()
    p.close()
    return c


def _around(hub, others, d):
    rng = np.random.default_rng(1)
    return make_gates([(KIND_U, 0, -1, haar_u2(rng))] + [(KIND_CU, hub, q, np.diag([1.0, d])) for q in others])


def test_phases_that_share_a_bit_are_counted_as_one_group():
    c = _counts(_around(0, range(1, 9), np.exp(0.3j)), 9, 9)
    assert c["fan"] == 1 and c["fan_phase"] == c["diag"] == 8
    # two are not worth a group
    c = _counts(_around(0, (5, 6), np.exp(0.3j)), 9, 9)
    assert c["fan"] == c["fan_phase"] == 0 and c["diag"] == 2


def test_factors_far_from_modulus_one_stay_on_their_own():
    for d in (1e25, 1e-25, 0.0, 2.0, np.inf, np.nan):
        c = _counts(_around(0, range(1, 9), d), 9, 9)
        assert c["fan"] == 0 and c["diag"] == 8


@pytest.mark.parametrize("n,k", [(13, 9), (13, 12), (22, 12), (30, 12)])
def test_fourier_transforms_run_their_phases_in_groups(n, k):
    c = _counts(qft_circuit(n), n, k)
    assert c["diag"] + c["dispatch"] == n * (n - 1) / 2
    assert c["fan"] > 0 and c["fan_phase"] > 0.5 * c["diag"]


def test_predictions_do_not_price_grouped_phases_as_diagonal_gates():
    cm = costmodel.CostModel("c128", n_cal=24)
    cm.launch_costs = {c: 0.0 for c in ("plain_u", "plain_cu", "plain_cx", "plain_cz", "move", "move_fraction")}
    cm.tile_costs = {(12, 0): {**dict.fromkeys(costmodel.TILE_CLASSES, 0.0), "diag": 1.0}}
    ms, c = cm.predict(qft_circuit(24), 24, k_tile=12, max_swaps=4, pinned=3, perm_exec="relabel")
    assert ms == c["diag"] - c["fan_phase"] < 0.5 * c["diag"]


def test_costs_without_the_classes_of_groups_price_phases_one_by_one():
    cm = costmodel.CostModel("c128", n_cal=24)
    cm.launch_costs = {c: 0.0 for c in ("plain_u", "plain_cu", "plain_cx", "plain_cz", "move", "move_fraction")}
    cm.tile_costs = {(12, 0): {c: 2.0 if c == "diag" else 0.0 for c in costmodel.TILE_CLASSES if "fan" not in c}}
    ms, c = cm.predict(qft_circuit(24), 24, k_tile=12, max_swaps=4, pinned=3, perm_exec="relabel")
    assert ms == 2.0 * c["diag"] and c["fan_phase"] > 0


@pytest.mark.parametrize("k", range(2, 15))
def test_calibration_circuits_of_every_tile(k):
    for log_r in range(1, 6):
        for dt in ("c64", "c128"):
            for name, g in costmodel.calibration_circuits(20, k, log_r).items():
                Q.Program(g, 20, dt, form="pass", k_tile=k, max_swaps=1, pinned=min(k, 3) - 1, perm_exec="relabel",
                          reg_bits=log_r).close()


@pytest.mark.parametrize("k,log_r", [(7, 1), (9, 3), (12, 4), (13, 5)])
def test_calibration_separates_groups_from_their_phases(k, log_r):
    rows = [costmodel.tile_work(_counts(g, 22, k, reg_bits=log_r, max_swaps=1, **costmodel.CAL_OPTS.get(name, {})))
            for name, g in costmodel.calibration_circuits(22, k, log_r).items()]
    a = np.array(rows)
    fan, spoke = (a[:, costmodel.TILE_CLASSES.index(c)] for c in ("fan", "fan_phase"))
    assert (spoke > 0).sum() == 2 and fan.max() >= 1.5 * fan[fan > 0].min()
    # every class that the shape has is determined
    used = a[:, a.any(axis=0)]
    assert np.linalg.matrix_rank(used) == used.shape[1]
