"""Controlled phases that share a bit run as one multiplication per pass
operation: the shared bit on a register slot, on a thread bit and outside the
tile, the other bits anywhere, in every tile shape, against the oracle."""

import math

import numpy as np
import pytest

import oracle as O
from workloads import KIND_CU, KIND_CX, KIND_U, haar_u2, make_gates, phase, qft_circuit

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402

TOL = {"c128": 1e-12, "c64": 1e-5}


def _hubs(n, seed):
    """Runs of 2 to n controlled phases around one qubit (as control or as target, a pair twice now and then, some
    with a first entry that is not 1), with one-qubit gates and CNOTs between the runs."""
    rng = np.random.default_rng(seed)
    recs = [(KIND_U, q, -1, haar_u2(rng)) for q in range(n)]
    for _ in range(12):
        hub = int(rng.integers(n))
        for q in rng.permutation(n)[: int(rng.integers(2, n + 1))]:
            q = int(q)
            if q == hub:
                continue
            m = phase(float(rng.uniform(0, 2 * math.pi)))
            if rng.uniform() < 0.1:
                m = np.diag(np.exp(1j * rng.uniform(0, 2 * math.pi, 2)))
            pair = (hub, q) if rng.uniform() < 0.5 else (q, hub)
            recs += [(KIND_CU, *pair, m)] * (2 if rng.uniform() < 0.1 else 1)
        a, b = (int(v) for v in rng.choice(n, 2, replace=False))
        recs += [(KIND_U, a, -1, haar_u2(rng)), (KIND_CX, a, b, None)]
    return make_gates(recs)


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,k,regs", [(9, 9, 0), (10, 7, 1), (12, 8, 2), (13, 9, 3), (13, 12, 2), (14, 11, 5), (15, 12, 4),
                                      (16, 10, 0)])
def test_fans_match_oracle(n, k, regs, dt):
    print("phase fans", n, k, regs, dt, flush=True)
    rng = np.random.default_rng(n)
    start = make_gates([(KIND_U, q, -1, haar_u2(rng)) for q in range(n)])
    for g in (np.concatenate([start, qft_circuit(n)]), _hubs(n, 7 * n + k)):
        ref = O.run(g, n)
        for pinned in (0, 3):
            opts = dict(form="pass", k_tile=k, max_swaps=4, pinned=pinned, perm_exec="relabel", reg_bits=regs)
            st = Q.State(n, dt).run(g, **opts)
            assert np.abs(st.to_numpy() - ref).max() <= TOL[dt]
            # the read-out folded into a last pass that holds fans
            st = Q.State(n, dt)
            assert np.abs(st.run_expect_z(g, **opts) - O.expect_z(ref, n)).max() <= TOL[dt]


def test_fans_in_batches_and_work_counts():
    n = 13
    circ = [(m, qft_circuit(m)) for m in (9, 12, n)]
    b = Q.Batch([(m, np.concatenate([make_gates([(KIND_U, 0, -1, haar_u2(np.random.default_rng(m)))]), g]))
                 for m, g in circ], "c128", k_tile=12, max_swaps=8)
    z, norm = b.run().results()
    assert np.abs(norm - 1).max() <= 1e-12
    b.close()
    # every controlled phase counted as one diagonal gate, or as skipped where its control outside the tile is 0
    p = Q.Program(qft_circuit(n), n, "c128", form="pass", k_tile=9, max_swaps=4, pinned=3, perm_exec="relabel")
    c = p.op_counts()
    p.close()
    assert c["diag"] + c["dispatch"] == n * (n - 1) / 2
