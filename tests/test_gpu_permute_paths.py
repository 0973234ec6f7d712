"""PermuteQubits on every route of the data movement: short cycles (tile
passes), the reversal (one involution), rotations and random placements (two
involutions), at sizes below, at and above the tiles.  Bit-exact against the
index map computed on the CPU."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402


def _placements(n):
    rng = np.random.default_rng(n)
    swap = list(range(n))
    swap[0], swap[n - 1] = swap[n - 1], swap[0]
    out = {"swap": swap, "reversal": list(range(n))[::-1], "rotation": [(q + 1) % n for q in range(n)],
           "rotation by 3 of the high ones": [q if q < 3 else 3 + (q - 3 + 2) % (n - 3) for q in range(n)] if n > 4 else swap}
    for i in range(3):
        out["random %d" % i] = [int(v) for v in rng.permutation(n)]
    return out


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 7, 8, 10, 11, 12, 13, 14, 15, 17, 19])
def test_move_is_exact(n, dt):
    print("permute", n, dt, flush=True)
    real, cplx = (np.float32, np.complex64) if dt == "c64" else (np.float64, np.complex128)
    a = np.random.default_rng(n).standard_normal(2 << n).astype(real)
    idx = np.arange(1 << n)
    for name, sigma in _placements(n).items():
        st = Q.State(n, dt)
        buf = st.buffer.view(torch.float32 if dt == "c64" else torch.float64)
        buf.copy_(torch.from_numpy(a))
        st.permute(sigma)
        j = np.zeros_like(idx)
        for q in range(n):
            j |= ((idx >> q) & 1) << sigma[q]
        want = np.empty(1 << n, dtype=cplx)
        want[j] = a.view(cplx)
        st.synchronize()
        assert np.array_equal(buf.cpu().numpy().view(cplx), want), name
        # and on from there: a composite of two moves, back to where it began
        st.permute(list(range(n))[::-1])
        st.permute(list(range(n)))
        st.synchronize()
        assert np.array_equal(buf.cpu().numpy(), a), name
