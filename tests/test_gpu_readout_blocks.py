"""Read-out sums at the edges of their blocks: one thread, one wavefront, one
block, the first sizes with several blocks, odd sizes above; every placement
of the second state of a fidelity.  Reference: the same sums in float64 by
torch on the amplitudes the states were given."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402

REAL = {"c64": torch.float32, "c128": torch.float64}


def _filled(n, dt, seed):
    """A state holding random amplitudes (identity placement), and those amplitudes in complex128."""
    st = Q.State(n, dt)
    x = torch.randn(2 << n, device="cuda", dtype=REAL[dt], generator=torch.Generator("cuda").manual_seed(seed))
    st.buffer.view(REAL[dt])[:] = x
    return st, torch.view_as_complex(x.double().view(-1, 2))


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 2, 6, 7, 8, 9, 11, 12, 13, 14, 15, 18, 21, 22])
def test_sums_at_block_edges(n, dt):
    print("read-out", n, dt, flush=True)
    a, x = _filled(n, dt, n)
    p = x.abs().square()
    norm = p.sum().item()
    z = [(v[:, 0].sum() - v[:, 1].sum()).item() for v in (p.view(-1, 2, 1 << q) for q in range(n))]
    # FP64 sums of 2^n non-negative terms in trees of at most 2^6 serial steps: 2^8 ulp
    tol = 2.0 ** -44 * norm
    assert np.abs(a.expect_z() - z).max() <= tol
    assert abs(a.norm() - norm) <= tol
    sigma = [int(v) for v in np.random.default_rng(n).permutation(n)]
    for other in ("c64", "c128"):
        b, y = _filled(n, other, 100 + n)
        want = 1.0 - abs(torch.vdot(x, y).item()) ** 2 / (norm * y.abs().square().sum().item())
        far = (x - y).abs().max().item()
        for place in (list(range(n)), sigma):
            b.permute(place)
            loss, diff = a.fidelity(b)
            assert abs(loss - want) <= 2.0 ** -42
            assert abs(diff - far) <= 2.0 ** -48 * far


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 10, 11, 19, 20, 21, 22])
def test_whole_state_in_logical_order(n, dt):
    print("whole state", n, dt, flush=True)
    a, x = _filled(n, dt, n)
    want = x.cpu().numpy()
    for sigma in (list(range(n)), list(range(n))[::-1], [int(v) for v in np.random.default_rng(n).permutation(n)]):
        a.permute(sigma)
        assert np.array_equal(a.to_numpy(), want)
