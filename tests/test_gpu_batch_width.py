"""Batches whose circuits have few tiles at a time: more workgroups per compute
unit must not slow them down.  Before waiting workgroups were bounded, four per
compute unit took 2.2 (complex128) and 3.2 times (complex64) as long as one here."""

import time

import numpy as np
import pytest

import oracle as O
from workloads import layered_circuit

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402


@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_more_workgroups_do_not_slow_narrow_batches(dt):
    print("narrow batch", dt, flush=True)
    rng = np.random.default_rng(16)
    circuits = [(int(n), layered_circuit(int(n), 30, int(n) + i)) for i, n in enumerate(rng.integers(10, 19, 16))]
    best = {}
    for wg in (1, 4):
        b = Q.Batch(circuits, dt, k_tile=11, max_swaps=8, pinned=4, wg_per_cu=wg, chunk=1, use_graph=0)
        z, norm = b.run().results()
        assert np.abs(norm - 1).max() <= (1e-4 if dt == "c64" else 1e-11)
        for _ in range(5):
            t = time.perf_counter()
            for _ in range(10):
                b.run()
            b.results()
            best[wg] = min(best.get(wg, 1e9), time.perf_counter() - t)
        b.close()
    n, g = circuits[0]
    assert abs(z[0] - O.expect_z(O.run(g, n), n)[0]) <= (1e-5 if dt == "c64" else 1e-12)
    assert best[4] <= 1.5 * best[1], best
