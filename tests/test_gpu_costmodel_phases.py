"""The cost model on circuits of controlled phases, which run in groups."""

import pytest

from workloads import qft_circuit

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import costmodel  # noqa: E402


@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_fourier_transform_is_predicted_within_a_factor_of_two(dt):
    n = 24
    cm = costmodel.CostModel(dt, n_cal=24)
    o = dict(k_tile=12, max_swaps=16, pinned=3, perm_exec="relabel", reg_bits=0)
    g = qft_circuit(n)
    predicted, _ = cm.predict(g, n, **o)
    measured = costmodel.measure_ms(g, n, dt, o, reps=5)
    print("qft", dt, predicted, measured, cm.tile_costs, flush=True)
    assert 0.5 < predicted / measured < 2.0
