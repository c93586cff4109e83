"""The gradient of given neighbour sets against the dense graph Laplacian in
FP64, shared by the backward's tests.

The kernel sums in FP64 and rounds once to FP32: 2^-24 of the value, plus FP64
rounding of at most (terms + 1) 2^-52 of the sum of the terms' magnitudes.
"""
import numpy as np
import torch


def bucket_lists(rng, n, k, w, sizes, at):
    """Neighbour lists idx [n, k] in which trajectory at[i] is a neighbour of the
    weighted trajectories exactly sizes[i] times; the other entries are -1."""
    idx = np.full(n * k, -1, dtype=np.int32)
    slots = rng.permutation(np.flatnonzero(np.repeat(w != 0.0, k)))[:sum(sizes)]
    assert len(slots) == sum(sizes)
    idx[slots] = np.repeat(np.asarray(at, dtype=np.int32), sizes)
    idx = idx.reshape(n, k)
    got = np.bincount(idx[w != 0.0].ravel() + 1, minlength=n + 1)[1:]
    assert np.array_equal(got[at], sizes) and got.sum() == sum(sizes)
    return idx


def check_gradient(T, D, L, k, idx, w, seed):
    from paper_2603_02059_amd import traknn as tk
    n = T - L + 1
    X = np.random.default_rng(seed).standard_normal((T, D)).astype(np.float32)
    xs = torch.zeros(T, (D + 3) // 4 * 4, device="cuda")
    xs[:, :D] = torch.from_numpy(X)
    p = tk.Plan(T, D, L, L, k, "fp32")
    args = (xs[:, :D], torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda())
    g = p.backward(*args).cpu().numpy()
    assert np.array_equal(g, p.backward(*args).cpu().numpy())
    p.close()
    A, count = np.zeros((T, T)), np.zeros(T)
    t, q = np.nonzero((idx >= 0) & (idx < n) & (w != 0.0)[:, None])
    for m in range(L):
        np.add.at(A, (t + m, idx[t, q] + m), w[t] / k)
        np.add.at(count, t + m, 1)
        np.add.at(count, idx[t, q] + m, 1)
    A += A.T
    Xd = X.astype(np.float64)
    mag = 2.0 * (np.abs(A).sum(1)[:, None] * np.abs(Xd) + np.abs(A) @ np.abs(Xd))
    ref = 2.0 * (A.sum(1)[:, None] * Xd - A @ Xd)
    assert np.all(np.abs(g - ref) <= 2.0 ** -24 * np.abs(ref) + (count.max() + 1) * 2.0 ** -52 * mag)
    assert np.all(g[np.abs(A).sum(1) == 0] == 0)
