"""Distances that are +inf (a cell beyond FP16's range) are never listed: a row
without k finite candidates ends in index -1 and +inf, as the clamp of the
distances (dist_clamp.h) promises, in the first and the later rounds of the
window, in a sweep, in bands and in the fused mode.

A trajectory that holds the overflowing field has no finite distance at all. In
the matrix mode the sums of the rows after it, up to the end of their block of
eight rows, slide through it (inf - inf), so only the other blocks are expected
to be full.
"""
import numpy as np
import pytest

from paper_2603_02059_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,L,L_max,k,rb,mode", [
    (300, 1, 1, 10, 0, "matrix"), (300, 3, 3, 64, 0, "matrix"),   # one round, dense
    (1600, 3, 3, 1, 0, "matrix"), (1601, 5, 5, 64, 0, "matrix"),  # later rounds too
    (1100, 1, 10, 10, 0, "matrix"), (700, 1, 3, 64, 0, "matrix"),  # ten lengths a pass, and one
    (1545, 3, 3, 12, 328, "matrix"),                              # from running lists
    (300, 3, 3, 64, 0, "fused"), (1600, 1, 1, 10, 0, "fused"),    # one and more rounds of tiles
])
def test_infinite_distances_are_not_listed(T, L, L_max, k, rb, mode):
    from paper_2603_02059_amd import traknn as tk
    print(f"[gpu] overflow T={T} L={L}..{L_max} k={k} row_batch={rb} {mode}", flush=True)
    x = synth.random_fields(T, 20, T + k, scale=100.0)
    bad = T // 2 + 3
    x[bad, 7] = 1.0e6
    idx, dist = tk.knn(torch.from_numpy(x).cuda(), L, k, "fp16", L_max=L_max, row_batch=rb,
                       mode=mode)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    for q, l in enumerate(range(L, L_max + 1)):
        n = T - l + 1
        t = np.arange(n)
        i, d = idx[q, :n], dist[q, :n]
        assert np.array_equal(i < 0, np.isinf(d))
        holds = (t <= bad) & (t + l > bad)
        assert np.all(i[holds] == -1)
        clear = ~(holds if mode == "fused" else np.isin(t // 8, t[holds] // 8))
        assert np.all(i[clear] >= 0)
        assert not np.any((i <= bad) & (i + l > bad) & (i >= 0))
        assert np.all((np.abs(i - t[:, None]) >= l) | (i < 0))
