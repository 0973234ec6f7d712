"""The cost model prices a program by the tile shape it has: small states get
other register bits than large ones, and their costs are those of that shape
(host only: costs are given, not measured)."""

import pytest

from paper_2010_09746_amd import costmodel
from paper_2010_09746_amd import qsim as Q
from workloads import layered_circuit

OPTS = dict(k_tile=12, max_swaps=8, pinned=3, perm_exec="relabel")


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,k", [(8, 8), (10, 10), (12, 12), (14, 10), (16, 8), (20, 12), (21, 12), (22, 12), (24, 9)])
@pytest.mark.parametrize("reg_bits", [0, 2, 5])
def test_log_r_is_that_of_the_compiled_program(n, k, dt, reg_bits):
    g = layered_circuit(n, 10, n)
    o = dict(OPTS, form="pass", k_tile=k)

    def counts(rb):
        p = Q.Program(g, n, dt, **dict(o, reg_bits=rb))
        c = p.op_counts()
        p.close()
        return c

    log_r = costmodel.CostModel(dt)._log_r(k, reg_bits, n)
    assert counts(reg_bits) == counts(log_r)
    # the counts do tell shapes apart (6 thread bits at least: one or two shapes at 7 and 8)
    if k > 8:
        assert counts(log_r) != counts(log_r - 1 if log_r > k - 10 and log_r > 1 else log_r + 1)


def _model(dt, **costs):
    cm = costmodel.CostModel(dt, n_cal=24)
    cm.launch_costs = {c: 0.0 for c in ("plain_u", "plain_cu", "plain_cx", "plain_cz", "move", "move_fraction")}
    cm.tile_costs = {shape: dict.fromkeys(costmodel.TILE_CLASSES, v) for shape, v in costs["tile_costs"].items()}
    return cm


@pytest.mark.parametrize("n,shape", [(16, (12, 3)), (21, (12, 3)), (22, (12, 0)), (26, (12, 0))])
def test_predictions_take_the_costs_of_the_shape(n, shape):
    cm = _model("c128", tile_costs={(12, 0): 1.0, (12, 3): 100.0})
    g = layered_circuit(n, 6, n)
    ms, counts = cm.predict(g, n, **OPTS)
    want = cm.tile_costs[shape]["u"] * 2.0 ** (n - 24) * (sum(counts[c] for c in costmodel.TILE_CLASSES)
                                                          + 0.5 * counts["phase"])
    assert abs(ms - want) <= 1e-9 * want
    assert cm.pass_costs(n, 12)["tile"] == 5 * cm.tile_costs[shape]["u"] * 2.0 ** (n - 24)
    best, table = cm.choose(g, n, ks=(12,), rs=(8,))
    assert abs(table[0]["predicted_ms"] - want) <= 1e-9 * want


def test_calibration_is_of_the_shape_it_names(monkeypatch):
    """Circuits of n_cal qubits, also where the library itself would give so few qubits another shape."""
    seen = []
    monkeypatch.setattr(costmodel, "_pass_ms", lambda st, prog, reps=3: seen.append(prog.op_counts()) or 1.0)
    cm = costmodel.CostModel("c128", n_cal=20)
    cm.calibrate_tile(None, 12, 0)
    by_default, seen = seen[:], []
    monkeypatch.setattr(costmodel, "_pass_ms", lambda st, prog, reps=3: seen.append(prog.op_counts()) or 1.0)
    cm.calibrate_tile(None, 12, 4)
    assert by_default == seen
    assert set(cm.tile_costs) == {(12, 0), (12, 4)}


def test_costs_brought_to_a_host_without_a_device(monkeypatch):
    """Nothing can measure the small state's shape there: the costs given for the options still price it."""
    monkeypatch.setattr(costmodel.torch.cuda, "is_available", lambda: False)
    cm = _model("c128", tile_costs={(12, 0): 1.0})
    ms, counts = cm.predict(layered_circuit(16, 6, 16), 16, **OPTS)
    assert ms > 0 and set(cm.tile_costs) == {(12, 0)}
    assert cm.choose(layered_circuit(16, 6, 16), 16, ks=(12,), rs=(8,))[1][0]["predicted_ms"] == ms
