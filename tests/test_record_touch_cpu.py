"""Which tile passes read their records ahead: those of few workgroups, and
those whose workgroups have wavefronts to share the table.  One wavefront would
read the whole of it for one tile, and many tiles at a time hide the misses."""

import ctypes

import numpy as np
import pytest

from host_runtime import host_library
from paper_2010_09746_amd import qsim as Q
from workloads import layered_circuit, paper_random_circuit


def _launches(L):
    a, b = ctypes.c_uint64(), ctypes.c_uint64()
    L.host_tile_launches(ctypes.byref(a), ctypes.byref(b))
    return a.value, b.value


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,k,ahead", [(8, 8, True), (14, 8, True), (18, 8, True), (19, 8, False), (20, 12, True),
                                       (20, 10, True), (20, 9, False), (21, 7, False), (22, 10, False),
                                       (22, 12, True), (23, 12, True)])
def test_states_run_by_themselves(n, k, ahead, dt):
    """Up to 2^10 tiles per pass, or 2^8 threads per tile (16 amplitudes each: tiles of 2^12)."""
    with host_library() as L:
        buf = np.zeros((2 << n) + 4, dtype=np.float32 if dt == "c64" else np.float64)
        buf = buf[(-buf.ctypes.data % 16) // buf.itemsize:][: 2 << n]
        st = Q.qs_state_create(n, dt, buf.ctypes.data, buf.nbytes, 0)
        # whole 128-byte lines
        o = Q.make_opts(k_tile=k, max_swaps=8, pinned=4 if dt == "c64" else 3, perm_exec="relabel")
        for g in (layered_circuit(n, 4, n), paper_random_circuit(n, 6 * n, 0.5, n)):
            p = Q.qs_compile(g, n, dt, None, o)
            passes = Q.qs_program_get_stats(p)["n_tile_passes"]
            _launches(L)
            Q.qs_run_program(st, p)
            assert _launches(L) == ((passes, 0) if ahead else (0, passes))
            Q.qs_run_circuit(st, g, o)
            assert _launches(L) == ((passes, 0) if ahead else (0, passes))
            Q.qs_program_destroy(p)
        Q.qs_state_destroy(st)


@pytest.mark.parametrize("n,k", [(12, 9), (21, 7), (21, 9)])
def test_passes_over_partial_lines_always_do(n, k):
    with host_library() as L:
        buf = np.zeros((2 << n) + 4, dtype=np.float32)
        buf = buf[(-buf.ctypes.data % 16) // 4:][: 2 << n]
        st = Q.qs_state_create(n, "c64", buf.ctypes.data, buf.nbytes, 0)
        # every qubit below the line leaves it by an exchange: no pass moves whole lines but the first
        o = Q.make_opts(k_tile=k, max_swaps=16, pinned=0, perm_exec="relabel")
        p = Q.qs_compile(layered_circuit(n, 6, n), n, "c64", None, o)
        passes = Q.qs_program_get_stats(p)["n_tile_passes"]
        _launches(L)
        Q.qs_run_program(st, p)
        ahead, others = _launches(L)
        assert ahead + others == passes and ahead >= passes - 2
        Q.qs_program_destroy(p)
        Q.qs_state_destroy(st)
