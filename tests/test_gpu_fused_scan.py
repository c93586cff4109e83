"""The FP64 fused mode's two filter consumers: a wave per recipient for small k,
the diagonal scan of both sides from k = 8 on. The k nearest are the first k of
the k + m nearest, so the lists of either must agree on their common part, bit
for bit; lengths at either end (the scan's diagonals per row block change with
L), widths around the 16-cell staging step, ragged last blocks, and a ramp, on
which whole tiles pass the bounds and overflow their slots.
"""
import numpy as np
import pytest

from paper_2603_02059_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["noise", "ramp"])
@pytest.mark.parametrize("T,D,L,k", [
    (700, 1, 1, 8), (1100, 15, 2, 9), (1500, 16, 5, 40), (1501, 17, 8, 64),
    (900, 33, 16, 10), (2600, 13, 4, 12),
])
def test_scan_equals_recipient_walk(kind, T, D, L, k):
    from paper_2603_02059_amd import traknn as tk
    print(f"[gpu] fused scan {kind} T={T} D={D} L={L} k={k}", flush=True)
    x = synth.random_fields(T, D, T + D, scale=100.0)
    if kind == "ramp":
        x = x + np.float32(7.0) * np.arange(T, dtype=np.float32)[:, None]
    X = torch.zeros(T, (D + 3) // 4 * 4, device="cuda")
    X[:, :D] = torch.from_numpy(x)
    X = X[:, :D]
    a, b = (tk.knn(X, L, q, "fp64", mode="fused") for q in (k, 7))
    assert torch.equal(a[0][..., :7], b[0]) and torch.equal(a[1][..., :7], b[1])
    n = T - L + 1
    idx, dist = a[0][0].cpu().numpy(), a[1][0].cpu().numpy()
    assert np.all(np.abs(idx - np.arange(n)[:, None]) >= L)
    assert np.all((dist[:, :-1] < dist[:, 1:]) |
                  ((dist[:, :-1] == dist[:, 1:]) & (idx[:, :-1] < idx[:, 1:])))
    # every list against direct FP64 distances: 2^-24 of each rounded snapshot
    # distance, and Eq. 4 in FP64 on centred fields
    xd = x.astype(np.float64)
    xc = xd - xd.mean(0)
    S = ((xc[:, None, :] - xc[None, :, :]) ** 2).sum(2) if D <= 17 and T <= 1200 else None
    if S is not None:
        Dm = sum(S[m:m + n, m:m + n] for m in range(L))
        off = np.abs(np.arange(n)[:, None] - np.arange(n)[None, :]) < L
        kth = np.sort(np.where(off, np.inf, Dm), axis=1)[:, :k]
        np.testing.assert_allclose(dist, kth, rtol=2.0 ** -23, atol=2.0 ** -40 * (xc * xc).sum(1).max())
