"""The gradient's stores: through the caches up to their 256 MB, past them for a
larger gradient, by element where its rows are not aligned. With the lists given
every column of the gradient is a sum of its own, so one gradient beyond 256 MB
has to equal, bit for bit, the gradients of its columns' parts, which stay below,
and the one with unaligned rows.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,D,L,k", [(4099, 16385, 2, 3), (5000, 13424, 4, 2)])
def test_gradient_stores_agree(T, D, L, k):
    from paper_2603_02059_amd import traknn as tk
    assert T * D * 4 > 256 << 20
    print(f"[gpu] gradient stores T={T} D={D}", flush=True)
    rng = np.random.default_rng(T)
    n = T - L + 1
    idx = torch.from_numpy(rng.integers(0, n, (n, k)).astype(np.int32)).cuda()
    w = rng.standard_normal(n)
    w[n // 3:n // 2] = 0.0
    w = torch.from_numpy(w).cuda()
    gen = torch.Generator(device="cuda").manual_seed(T)
    X = torch.randn(T, (D + 3) // 4 * 4, device="cuda", generator=gen)[:, :D]

    def grad(x, ldg):
        p = tk.Plan(T, x.shape[1], L, L, k, "fp32")
        p.release_workspace()
        buf = torch.full((T, ldg), float("nan"), device="cuda")
        g = p.backward(x, idx, w, buf[:, :x.shape[1]])
        p.close()
        assert bool(torch.isnan(buf[:, x.shape[1]:]).all())
        return g

    whole = grad(X, (D + 7) // 4 * 4)
    assert torch.equal(whole, grad(X, D + (D % 4 == 0)))
    half = D // 8 * 4
    assert torch.equal(whole[:, :half], grad(X[:, :half], half))
    assert torch.equal(whole[:, half:], grad(X[:, half:], (D - half + 7) // 4 * 4))
