"""Controlled phases in batches, where each runs as an operation of its own:
<Z_0> of circuits in which it depends on the phases, against the oracle."""

import math

import numpy as np
import pytest

import oracle as O
from workloads import KIND_CU, KIND_U, H, haar_u2, make_gates, phase, qft_circuit

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402

TOL = {"c128": 1e-12, "c64": 1e-5}


def _circuits():
    out = []
    for n in (9, 11, 12, 14):
        rng = np.random.default_rng(n)
        start = make_gates([(KIND_U, q, -1, haar_u2(rng)) for q in range(n)])
        around = [(KIND_CU, 0, q, phase(float(rng.uniform(0, 2 * math.pi)))) for q in range(1, n)]
        end = make_gates([(KIND_U, 0, -1, H)])
        out.append((n, np.concatenate([start, make_gates(around), end])))
        out.append((n, np.concatenate([start, qft_circuit(n)])))
    return out


@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_phases_in_a_batch(dt):
    circuits = _circuits()
    b = Q.Batch(circuits, dt, k_tile=12, max_swaps=8)
    z, norm = b.run().results()
    b.close()
    for c, (n, g) in enumerate(circuits):
        want = O.expect_z(O.run(g, n), n)[0]
        assert abs(z[c] - want) <= TOL[dt] and abs(norm[c] - 1) <= TOL[dt]
        # without the phases it is another number
        bare = g[g["kind"] != KIND_CU]
        assert abs(O.expect_z(O.run(bare, n), n)[0] - want) > 1e-3
