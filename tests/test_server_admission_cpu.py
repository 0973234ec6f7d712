"""qs_server_admit with programs of small states, which it compiles for the
server's tile shape: a refusal costs no compile, and a program is compiled for
servers once, however often and from however many threads it is admitted."""

import threading
import time

import numpy as np
import pytest

from host_runtime import host_library
from paper_2010_09746_amd import qsim as Q
from workloads import layered_circuit, mixed_circuit

N = 14


def _server(**kw):
    o = Q.make_batch_opts(**{**dict(k_tile=10, max_swaps=8, pinned=3, chunk=4, wg_per_cu=4, use_graph=0), **kw})
    return Q.qs_server_create("c64", o, 1 << 30, 8, 16)


def _program(gates, **kw):
    o = Q.make_opts(**{**dict(k_tile=10, max_swaps=8, pinned=3, perm_exec="relabel"), **kw})
    return Q.qs_compile(gates, N, "c64", None, o)


def _timed(f):
    t = time.perf_counter()
    try:
        got = f()
    except Q.QsimError as e:
        got = e.code
    return time.perf_counter() - t, got


def test_refusals_compile_nothing_and_admissions_compile_once():
    with host_library():
        srv, other = _server(), _server(reg_bits=2)
        compile_s, p = _timed(lambda: _program(mixed_circuit(N, 30000, 1)))
        buf = np.zeros(1 << N, dtype=np.complex64)
        none = np.zeros(0, dtype=np.uint64)
        admit = lambda s, size=8 << N, smp=none: _timed(lambda: Q.qs_server_admit(s, p, buf.ctypes.data, size, smp))
        small = Q.qs_server_create("c64", Q.make_batch_opts(k_tile=10, max_swaps=8, pinned=3, chunk=4, wg_per_cu=4,
                                                            use_graph=0), 1 << 10, 8, 16)
        for again in range(2):
            for code, (s, got) in ((-1, admit(srv, 8)), (-1, admit(srv, 8 << N, np.array([1 << N], dtype=np.uint64))),
                                   (-3, admit(small)), (-1, admit(other))):
                assert got == code
                assert s < 0.2 * compile_s
        first, got = admit(srv)
        assert got > 0
        for _ in range(3):
            s, got = admit(srv)
            assert got > 0
            assert s < 0.2 * compile_s
        for s in (srv, other, small):
            Q.qs_server_destroy(s)
        Q.qs_program_destroy(p)


def test_admissions_of_one_program_from_several_threads():
    with host_library():
        servers = [_server() for _ in range(4)]
        p = _program(layered_circuit(N, 30, 2))
        bufs = [np.zeros(1 << N, dtype=np.complex64) for _ in servers]
        got = [None] * len(servers)

        def one(i):
            got[i] = Q.qs_server_admit(servers[i], p, bufs[i].ctypes.data, 8 << N, np.zeros(0, dtype=np.uint64))

        ts = [threading.Thread(target=one, args=(i,)) for i in range(len(servers))]
        [t.start() for t in ts]
        [t.join() for t in ts]
        assert got == [1] * len(servers)
        for s in servers:
            Q.qs_server_destroy(s)
        Q.qs_program_destroy(p)


@pytest.mark.parametrize("kw,code", [(dict(k_tile=9), -1), (dict(reg_bits=2), -1), (dict(perm_exec="move"), -1),
                                     (dict(reg_bits=4), 1), (dict(), 1)])
def test_tile_options_that_a_server_takes(kw, code):
    with host_library():
        srv, p = _server(), _program(layered_circuit(N, 12, 3), **kw)
        buf = np.zeros(1 << N, dtype=np.complex64)
        assert _timed(lambda: Q.qs_server_admit(srv, p, buf.ctypes.data, 8 << N, np.zeros(0, dtype=np.uint64)))[1] == code
        Q.qs_server_destroy(srv)
        Q.qs_program_destroy(p)
