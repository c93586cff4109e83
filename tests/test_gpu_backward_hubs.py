"""The backward's reverse lists and row gather where they are long: a trajectory
that is a neighbour of 2, 64, 65, 1024, 1025 or nearly all others (its reverse
list is sorted in registers, in LDS or in place), rows with more terms than are
listed at once, zero weights, and odd widths. The lists are made up (the
gradient takes any neighbour sets), the reference is the dense graph Laplacian
in FP64, and two runs must agree bit for bit.

The kernel sums in FP64 and rounds once to FP32: 2^-24 of the value, plus FP64
rounding of at most (terms + 1) 2^-53 of the sum of the terms' magnitudes.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,D,L,k,hubs", [
    (300, 7, 1, 2, (2, 64)),
    (300, 12, 3, 2, (65, 200)),
    (1500, 5, 2, 3, (1024, 63)),
    (1500, 6, 4, 2, (1025, 130)),
    (2600, 1030, 5, 2, (2500, 64)),
])
def test_reverse_lists_of_hubs(T, D, L, k, hubs):
    from paper_2603_02059_amd import traknn as tk
    print(f"[gpu] hubs T={T} D={D} L={L} k={k} {hubs}", flush=True)
    rng = np.random.default_rng(T + D)
    n = T - L + 1
    X = rng.standard_normal((T, D)).astype(np.float32)
    idx = np.stack([(np.arange(n) + 7 + 13 * q) % n for q in range(k)], 1).astype(np.int32)
    for col, size in enumerate(hubs):
        rows = rng.permutation(n)[:size]
        idx[rows, col] = (3, n - 2)[col]
    w = rng.standard_normal(n)
    w[rng.permutation(n)[:n // 10]] = 0.0
    xs = torch.zeros(T, (D + 3) // 4 * 4, device="cuda")
    xs[:, :D] = torch.from_numpy(X)
    p = tk.Plan(T, D, L, L, k, "fp32")
    args = (xs[:, :D], torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda())
    g = p.backward(*args).cpu().numpy()
    assert np.array_equal(g, p.backward(*args).cpu().numpy())
    p.close()
    A = np.zeros((T, T))
    for m in range(L):
        np.add.at(A, (np.repeat(np.arange(n), k) + m, idx.reshape(-1) + m), np.repeat(w / k, k))
    A += A.T
    Xd = X.astype(np.float64)
    ref = 2.0 * (A.sum(1)[:, None] * Xd - A @ Xd)
    mag = 2.0 * (np.abs(A).sum(1)[:, None] * np.abs(Xd) + np.abs(A) @ np.abs(Xd))
    terms = 2 * L * n
    assert np.all(np.abs(g - ref) <= 2.0 ** -24 * np.abs(ref) + (terms + 1) * 2.0 ** -52 * mag)
    assert np.all(g[np.abs(A).sum(1) == 0] == 0)
