"""A served request's read-out where its buffer begins at an odd amplitude
(complex64: 8-byte, not 16-byte alignment): the same numbers as in an aligned
buffer, bit for bit."""

import numpy as np
import pytest

from workloads import layered_circuit, sample_indices

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402


@pytest.mark.parametrize("n", [10, 13, 14, 18])
def test_requests_at_any_amplitude(n):
    print("server buffer", n, flush=True)
    opts = Q.make_batch_opts(k_tile=10, max_swaps=8, pinned=3, chunk=4, wg_per_cu=4, use_graph=0)
    h = Q.qs_server_create("c64", opts, 1 << 30, 4, 16)
    idx = sample_indices(n, 16, n)
    with_reg = Q.Program(layered_circuit(n, 4, n), n, "c64", form="pass", k_tile=10, max_swaps=8, pinned=3,
                         perm_exec="relabel", reg_bits=4)
    res = []
    for at in (0, 1):
        buf = torch.empty((1 << n) + 1, dtype=torch.complex64, device="cuda")
        assert buf.data_ptr() % 16 == 0
        sid = Q.qs_server_admit(h, with_reg.h, buf.data_ptr() + 8 * at, 8 << n, idx)
        done = []
        while not done:
            Q.qs_server_step_launch(h)
            done = Q.qs_server_step_wait(h)
        z, amps, norm = Q.qs_server_result(h, sid, n, 16)
        Q.qs_server_release(h, sid)
        state = buf[at:at + (1 << n)].cpu().numpy()
        prob = np.abs(state.astype(np.complex128)) ** 2
        assert abs(norm - prob.sum()) <= 1e-12  # FP64 sums of at most 2^18 terms
        res.append((z, amps, norm))
    assert res[0][2] == res[1][2]
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])
    with_reg.close()
    Q.qs_server_destroy(h)
