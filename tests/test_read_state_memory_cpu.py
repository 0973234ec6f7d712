"""qs_read_state where the device has no room for its workspace, where an
allocation fails for another reason, and where another device is current: the
state still comes out, as it does without any workspace, and errors that are
not a lack of memory are reported at once."""

import contextlib

import numpy as np
import pytest

from host_runtime import host_library
from paper_2010_09746_amd import qsim as Q


@contextlib.contextmanager
def _state(n, dt, seed):
    """A state of random amplitudes under a random placement: its handle and its amplitudes in logical order and FP64."""
    rng = np.random.default_rng(seed)
    real, cplx = (np.float32, np.complex64) if dt == "c64" else (np.float64, np.complex128)
    buf = np.zeros((2 << n) + 4, dtype=real)
    buf = buf[(-buf.ctypes.data % 16) // buf.itemsize:][: 2 << n]
    h = Q.qs_state_create(n, dt, buf.ctypes.data, buf.nbytes, 0)
    sigma = [int(q) for q in rng.permutation(n)]
    Q.qs_permute_qubits(h, sigma)
    buf[:] = rng.standard_normal(2 << n)  # as stored under sigma
    j = np.zeros(1 << n, dtype=np.int64)
    for q in range(n):
        j |= ((np.arange(1 << n) >> q) & 1) << sigma[q]
    yield h, buf.view(cplx)[j].astype(np.complex128)
    Q.qs_state_destroy(h)


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("room", [1 << 30, 1 << 20, 16 << 10, 1024, 0])
@pytest.mark.parametrize("n", [5, 12, 17])
def test_any_room_on_the_device(n, room, dt):
    with host_library() as L:
        with _state(n, dt, n) as (h, want):
            L.host_set_budget(room)
            assert np.array_equal(Q.qs_read_state(h, n), want)
            assert L.host_used() <= min(room, 16 << 20)
            L.host_set_budget(2 ** 64 - 1)
        assert L.host_used() == 0


def test_other_errors_are_not_taken_for_a_lack_of_memory():
    with host_library() as L, _state(12, "c64", 1) as (h, want):
        L.host_set_malloc_error(719)  # a launch failure reported late
        before = L.host_mallocs()
        with pytest.raises(Q.QsimError) as e:
            Q.qs_read_state(h, 12)
        assert e.value.code == -4 and L.host_mallocs() == before + 1
        L.host_set_malloc_error(0)
        assert np.array_equal(Q.qs_read_state(h, 12), want)


def test_another_current_device():
    with host_library() as L, _state(10, "c64", 2) as (h, want):
        L.host_set_device(1)
        assert np.array_equal(Q.qs_read_state(h, 10), want)
        assert L.host_used() == 0
        L.host_set_device(0)


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,launches", [(1, False), (7, False), (8, True), (13, True)])
def test_few_amplitudes_are_ordered_by_the_host(n, launches, dt):
    with host_library() as L, _state(n, dt, n) as (h, want):
        assert np.array_equal(Q.qs_read_state(h, n), want)
        assert (L.host_used() > 0) == launches  # the workspace that the device's part of the work needs
