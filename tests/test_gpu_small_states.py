"""States of up to 2^21 amplitudes run with more threads per tile: the same
results as with the usual shape on both sides of that line, and programs
compiled for them still serve where one shape is shared."""

import numpy as np
import pytest

import oracle as O
from workloads import layered_circuit, mixed_circuit, sample_indices

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402
from paper_2010_09746_amd.serving import Server  # noqa: E402

TOL = {"c128": 1e-12, "c64": 1e-5}


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,k", [(7, 7), (8, 7), (9, 9), (10, 8), (12, 12), (13, 12), (14, 13), (15, 10), (16, 14)])
def test_small_states_match_oracle(n, k, dt):
    print("small state", n, k, dt, flush=True)
    for g in (layered_circuit(n, 4, n), mixed_circuit(n, 80, n)):
        ref = O.run(g, n)
        for perm_exec in ("relabel", "move"):
            opts = dict(form="pass", k_tile=k, max_swaps=4, pinned=2, perm_exec=perm_exec)
            assert np.abs(Q.State(n, dt).run(g, **opts).to_numpy() - ref).max() <= TOL[dt]
            p = Q.Program(g, n, dt, **opts)
            for noalloc in (False, True):
                assert np.abs(Q.State(n, dt).run_program(p, noalloc=noalloc).to_numpy() - ref).max() <= TOL[dt]


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [20, 21, 22])
def test_shapes_agree_around_the_line(n, dt):
    print("shape line", n, dt, flush=True)
    g, idx = layered_circuit(n, 6, n), sample_indices(n, 512, n)
    opts = dict(form="pass", k_tile=12, max_swaps=8, pinned=4, perm_exec="relabel")
    a = Q.State(n, dt).run(g, **opts)
    b = Q.State(n, dt).run(g, reg_bits=4, **opts)
    # amplitudes are about 2^(-n/2)
    tol = (1e-12 if dt == "c128" else 1e-4) * 2.0 ** (-n / 2)
    assert np.abs(a.amplitudes(idx) - b.amplitudes(idx)).max() <= tol
    assert a.sigma == b.sigma


def test_server_takes_programs_of_small_states():
    """A server's shared launch has one shape; programs compiled without reg_bits are taken whatever shape they have
    by themselves, programs with other explicit reg_bits are refused."""
    srv = Server("c64", k_tile=10, max_swaps=8, pinned=3, max_slots=8)
    reqs = [dict(id=i, arrival=0.0, n=n, gates=layered_circuit(n, 3, i), samples=sample_indices(n, 16, i))
            for i, n in enumerate((10, 12, 13, 15))]
    srv.compile = lambda g, n: Q.Program(g, n, "c64", form="pass", k_tile=10, max_swaps=8, pinned=3,
                                         perm_exec="relabel")
    res, _ = srv.serve(reqs, realtime=False)
    for r in reqs:
        ref = O.run(r["gates"], r["n"])
        assert np.abs(res[r["id"]]["amps"] - ref[np.asarray(r["samples"], dtype=np.int64)]).max() <= 1e-5
        assert np.abs(res[r["id"]]["z"] - O.expect_z(ref, r["n"])).max() <= 1e-5
    srv.compile = lambda g, n: Q.Program(g, n, "c64", form="pass", k_tile=10, max_swaps=8, pinned=3,
                                         perm_exec="relabel", reg_bits=3)
    with pytest.raises(Q.QsimError) as e:
        srv.serve(reqs[:1], realtime=False)
    assert e.value.code == -1
    srv.close()
