"""Programs of small states that would pass the record limit of the
allocation-free run in the shape of small states: they get the usual shape, at
the price of one compile."""

import time

import pytest

from paper_2010_09746_amd import qsim as Q
from workloads import layered_circuit, mixed_circuit

OPTS = dict(form="pass", k_tile=12, max_swaps=16, pinned=3, perm_exec="relabel")


def _compiled(g, n, **kw):
    t = time.perf_counter()
    p = Q.Program(g, n, "c128", **{**OPTS, **kw})
    t = time.perf_counter() - t
    got = (p.op_counts(), p.instructions(), {k: v for k, v in p.stats().items() if k != "compile_ms"})
    p.close()
    return t, got


@pytest.mark.parametrize("perm_exec", ["relabel", "move"])
@pytest.mark.parametrize("n,g", [(16, layered_circuit(16, 3000, 1)), (13, mixed_circuit(13, 40000, 2))])
def test_past_the_limit_the_program_is_that_of_the_usual_shape(n, g, perm_exec):
    kw = dict(perm_exec=perm_exec, max_swaps=16 if perm_exec == "relabel" else 1)
    assert _compiled(g, n, **kw)[1] == _compiled(g, n, reg_bits=4, **kw)[1]


def test_within_the_limit_it_is_not():
    g = layered_circuit(16, 100, 1)
    assert _compiled(g, 16)[1] == _compiled(g, 16, reg_bits=3)[1] != _compiled(g, 16, reg_bits=4)[1]


def test_it_costs_one_compile():
    g = layered_circuit(21, 6000, 1)
    usual = min(_compiled(g, 21, reg_bits=4)[0] for _ in range(2))
    assert min(_compiled(g, 21)[0] for _ in range(2)) < 1.5 * usual
