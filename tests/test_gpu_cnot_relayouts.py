"""CNOTs carried out by the write addresses of the next register re-layout:
chains that share targets and controls, controls on register slots and on
thread bits (more of them than one re-layout takes), in every register shape
and over wavefront-local re-layouts, against the oracle."""

import numpy as np
import pytest

import oracle as O
from workloads import KIND_CX, KIND_U, haar_u2, make_gates, paper_random_circuit, qft_like_circuit

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402

TOL = {"c128": 1e-12, "c64": 1e-5}


def _chains(n, seed):
    """Bursts of CNOTs (fans into one target, fans out of one control, chains, random) between a few one-qubit gates."""
    rng = np.random.default_rng(seed)
    recs = []
    for _ in range(8):
        p = [int(v) for v in rng.permutation(n)]
        kind = rng.integers(4)
        if kind == 0:
            recs += [(KIND_CX, c, p[0], None) for c in p[1:]]
        elif kind == 1:
            recs += [(KIND_CX, p[0], t, None) for t in p[1:]]
        elif kind == 2:
            recs += [(KIND_CX, a, b, None) for a, b in zip(p, p[1:])]
        else:
            recs += [(KIND_CX, *(int(v) for v in rng.choice(n, 2, replace=False)), None) for _ in range(n)]
        recs += [(KIND_U, q, -1, haar_u2(rng)) for q in p[: int(rng.integers(0, 4))]]
    return make_gates(recs)


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,k,regs", [(8, 8, 0), (9, 8, 1), (11, 9, 2), (12, 12, 3), (13, 10, 4), (14, 12, 4), (14, 13, 5),
                                      (16, 12, 0)])
def test_cnots_in_relayouts_match_oracle(n, k, regs, dt):
    print("cnots in re-layouts", n, k, regs, dt, flush=True)
    rng = np.random.default_rng(n)
    start = make_gates([(KIND_U, q, -1, haar_u2(rng)) for q in range(n)])
    absorbed = 0
    for g in (_chains(n, n), _chains(n, 3 * n), paper_random_circuit(n, 20 * n, 1.0, n),
              paper_random_circuit(n, 20 * n, 0.6, n), qft_like_circuit(n)):
        g = np.concatenate([start, g])
        ref = O.run(g, n)
        for flags in (dict(), dict(full_matrices=True)):
            opts = dict(form="pass", k_tile=k, max_swaps=4, pinned=2, perm_exec="relabel", reg_bits=regs, **flags)
            st = Q.State(n, dt).run(g, **opts)
            assert np.abs(st.to_numpy() - ref).max() <= TOL[dt]
            if n == k:  # no CNOT has its control outside the tile: every dispatch is a CNOT of a re-layout
                p = Q.Program(g, n, dt, **opts)
                absorbed += p.op_counts()["dispatch"]
                p.close()
    if n == k:
        assert absorbed > 0
    # a batch of the same circuits
    if n >= 9:
        gs = [(n, np.concatenate([start, _chains(n, s)])) for s in range(3)]
        b = Q.Batch(gs, dt, k_tile=max(9, min(k, 12)), max_swaps=4)
        z, norm = b.run().results()
        for c, (_, g) in enumerate(gs):
            assert abs(z[c] - O.expect_z(O.run(g, n), n)[0]) <= TOL[dt]
        b.close()
