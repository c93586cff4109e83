"""The sort of the reverse lists at its edges: up to 64 entries in registers, up
to 1024 in LDS, longer ones where they are. The lengths are exact (checked here
on the host), one short of each edge, on it and one past it.

The order shows in the sums: of a trajectory's reverse terms, by t, the first two
thirds are +2^60, -2^60 in turn and the others 1. Every field difference is 1 and
k a power of two, so in order the sum is exactly the number of ones, and a one
ahead of its turn is lost between 2^60 and -2^60.
"""
import numpy as np
import pytest

from tests.gradref import bucket_lists, check_gradient

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [2, 3, 63, 64, 65, 127, 1023, 1024, 1025, 1026, 2047]


@pytest.mark.parametrize("size", SIZES)
def test_reverse_list_order(size):
    from paper_2603_02059_amd import traknn as tk
    print(f"[gpu] reverse list of {size}", flush=True)
    T, D, k, hub = 2100, 4, 4, 1001
    rng = np.random.default_rng(size)
    ts = np.sort(rng.permutation(np.delete(np.arange(T), hub))[:size])
    idx = np.full((T, k), -1, dtype=np.int32)
    idx[ts, rng.integers(0, k, size)] = hub
    w = np.zeros(T)
    big = size // 3 * 2
    w[ts] = 1.0
    w[ts[:big:2]], w[ts[1:big:2]] = 2.0 ** 60, -2.0 ** 60
    assert np.bincount(idx[w != 0.0].ravel() + 1, minlength=T + 1)[1 + hub] == size
    X = torch.zeros(T, D, device="cuda")
    X[hub] = 1.0
    p = tk.Plan(T, D, 1, 1, k, "fp32")
    g = p.backward(X, torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda())
    p.close()
    assert g[hub].tolist() == [2.0 * (size - big) / k] * D


@pytest.mark.parametrize("L,D", [(1, 5), (3, 1030)])
def test_reverse_lists_of_exact_lengths(L, D):
    print(f"[gpu] reverse lists L={L} D={D}", flush=True)
    T, k = 2600, 5
    rng = np.random.default_rng(L)
    n = T - L + 1
    w = rng.standard_normal(n)
    w[rng.permutation(n)[:n // 10]] = 0.0
    idx = bucket_lists(rng, n, k, w, SIZES, 17 + 230 * np.arange(len(SIZES)))
    check_gradient(T, D, L, k, idx, w, L)
