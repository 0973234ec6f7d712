"""Data movement of small states: bit-exact where the tiles of an involution
grow with the state, and about as long as its launches."""

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no HIP device", allow_module_level=True)

from paper_2010_09746_amd import qsim as Q  # noqa: E402

REAL = {"c64": torch.float32, "c128": torch.float64}


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [14, 16, 18, 20, 21, 22, 23])
def test_moves_are_exact_at_every_tile_size(n, dt):
    print("permute", n, dt, flush=True)
    a = torch.randn(2 << n, dtype=REAL[dt], device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    amps, idx = torch.view_as_complex(a.view(-1, 2)), torch.arange(1 << n, device="cuda")
    rng = np.random.default_rng(n)
    for sigma in (list(range(n))[::-1], [(q + 1) % n for q in range(n)], [(q + n // 2) % n for q in range(n)],
                  [int(q) for q in rng.permutation(n)], [int(q) for q in rng.permutation(n)]):
        st = Q.State(n, dt)
        st.buffer.view(REAL[dt]).copy_(a)
        st.permute(sigma)
        j = torch.zeros_like(idx)
        for q in range(n):
            j |= ((idx >> q) & 1) << sigma[q]
        want = torch.empty_like(amps)
        want[j] = amps
        st.synchronize()
        assert torch.equal(torch.view_as_complex(st.buffer.view(REAL[dt]).view(-1, 2)), want)
        st.close()


@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_two_launches_take_no_longer_than_three_exchanges(dt):
    """16 qubits: a random placement (two involutions) against one exchanged pair (one pass).  With the tiles of large
    states, of which so small a state has sixteen, it took 4.3 times as long in complex64."""
    n = 16
    st, best = Q.State(n, dt), {}
    identity = list(range(n))
    rnd = [int(q) for q in np.random.default_rng(n).permutation(n)]
    pair = [n - 1] + identity[1:-1] + [0]
    for name, sigma in (("random", rnd), ("pair", pair)) * 4:
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(200):
            st.permute(sigma)
            st.permute(identity)
        torch.cuda.synchronize()
        best[name] = min(best.get(name, 1e9), time.perf_counter() - t)
    print(dt, best, flush=True)
    assert best["random"] <= 3 * best["pair"], best
