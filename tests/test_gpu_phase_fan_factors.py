"""Controlled phases whose factors are far from modulus 1 (gates need not be
unitary): the products of factors that no amplitude meets must not leave the
range of the type.  Reference: the same gates in one launch each."""

import numpy as np
import pytest

from workloads import KIND_CU, KIND_U, H, make_gates

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402


@pytest.mark.parametrize("dt,big", [("c64", 1e25), ("c128", 1e200)])
@pytest.mark.parametrize("hub", [0, 6, 11])  # a register slot or thread bit of the tile, outside it
def test_unused_products_stay_out_of_the_amplitudes(dt, big, hub):
    n, k = 12, 10
    print("fan factors", dt, hub, flush=True)
    partners = [q for q in range(n) if q != hub]
    start = [(KIND_U, q, -1, H) for q in range(n) if q == hub or q % 3 == 0]
    # the hub's partners are 0, so every amplitude keeps its value
    idle = [q for q in partners if q % 3]
    for d in (big, 1.0 / big, 0.0):
        g = make_gates(start + [(KIND_CU, hub, q, np.diag([1.0, d])) for q in idle])
        want = Q.State(n, dt).run(g, form="plain").to_numpy()
        assert np.isfinite(want).all() and abs(np.vdot(want, want) - 1) < 1e-5
        got = Q.State(n, dt).run(g, form="pass", k_tile=k, max_swaps=4, perm_exec="relabel").to_numpy()
        # the same Hadamards in another order: a few roundings apart
        assert np.abs(got - want).max() <= (1e-5 if dt == "c64" else 1e-13)
