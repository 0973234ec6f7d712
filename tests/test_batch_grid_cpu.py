"""Workgroups of a batch's launch: the caller's bound where the circuits have
work for them, fewer where most would wait."""

import pytest

from host_runtime import host_library
from paper_2010_09746_amd import qsim as Q
from workloads import layered_circuit

CUS = 256  # of the host runtime


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("sizes,k,per_cu", [([9], 9, 1), ([17], 9, 1), ([18], 9, 1), ([18, 12], 9, 2), ([19], 9, 2),
                                            ([20, 9], 9, 5), ([20], 9, 4), ([20] * 4, 9, 16)])
@pytest.mark.parametrize("asked", [0, 1, 3, 5])
def test_workgroups_by_the_items_that_can_run(sizes, k, per_cu, dt, asked):
    """One workgroup per compute unit for each two items per compute unit that the widest level has, begun or whole."""
    with host_library() as L:
        o = Q.make_batch_opts(k_tile=k, max_swaps=4, pinned=3, wg_per_cu=asked, chunk=1, use_graph=0)
        circuits = [(n, layered_circuit(n, 4, n)) for n in sizes]
        passes, items = Q.qs_batch_plan(circuits, dt, o)
        h = Q.qs_batch_create(circuits, dt, o)
        Q.qs_batch_run(h)
        assert L.host_queue_grid() == min(len(items), CUS * min(per_cu, asked or 4))
        Q.qs_batch_destroy(h)
        assert L.host_used() == 0
