"""The window stage's rounds: eight chunks of 64 diagonals a round, the few
candidates below a row's bound through LDS buffers, whole rounds densely where
they do not fit.

Two kinds of series force the dense rounds: noise (the first round, without a
bound) and a ramp, on which distances fall along the scan towards a row and so
every later round passes more candidates than a buffer holds. The fused mode
forms the same distances and selects them by other kernels, and the window sums
of these inputs are exact in both, so the lists must be equal; a sweep's passes
of ten, five, two and one lengths must equal the single lengths.
"""
import numpy as np
import pytest

from paper_2603_02059_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _series(kind, T, D, seed):
    x = synth.make_fields(T, 1, D, sigma=2.0, n_events=1, event_len=3, seed=seed)[0]
    if kind == "ramp":
        x = x + 300.0 * np.arange(T, dtype=np.float32)[:, None]
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


@pytest.mark.parametrize("kind", ["noise", "ramp"])
@pytest.mark.parametrize("T,L,k", [
    (513, 1, 10), (520, 16, 64),     # around one round of 512 diagonals
    (1030, 5, 64), (1545, 5, 10),    # two and three rounds, a ragged last block
    (1500, 1, 1), (4200, 3, 40),
])
def test_window_equals_fused(kind, T, L, k):
    from paper_2603_02059_amd import traknn as tk
    print(f"[gpu] window {kind} T={T} L={L} k={k}", flush=True)
    X = _series(kind, T, 50, T + L)
    a, b = tk.knn(X, L, k), tk.knn(X, L, k, mode="fused")
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("kind", ["noise", "ramp"])
@pytest.mark.parametrize("T,L_max,k,rb", [
    (1500, 10, 10, 0),    # one pass of ten lengths
    (1100, 16, 12, 0),    # ten, five and one
    (1545, 13, 20, 0),    # five, five, two and one
    (700, 3, 64, 0),      # one length a pass
    (1545, 12, 10, 328),  # the same from running lists, in bands
])
def test_sweep_passes_equal_single_lengths(kind, T, L_max, k, rb):
    from paper_2603_02059_amd import traknn as tk
    print(f"[gpu] sweep {kind} T={T} L_max={L_max} k={k} row_batch={rb}", flush=True)
    X = _series(kind, T, 50, T + k)
    idx, dist = tk.knn(X, 1, k, L_max=L_max, row_batch=rb)
    for L in range(1, L_max + 1):
        n = T - L + 1
        i1, d1 = tk.knn(X, L, k)
        assert torch.equal(idx[L - 1, :n], i1[0]) and torch.equal(dist[L - 1, :n], d1[0]), L
        assert bool((idx[L - 1, n:] == -1).all()) and bool(torch.isinf(dist[L - 1, n:]).all())
