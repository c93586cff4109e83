"""The rows of the gradient by their number of terms, where the gather changes
its ways: up to 8 terms of a row of L = 1 are read where they are, the first wave
lists a row's first 64 reverse terms, the whole workgroup the later ones, 256 at
a time. Rows without weight (no forward terms), missing neighbours (-1) and ones
beyond the series are among them; odd widths and more than one column block.
"""
import numpy as np
import pytest

from tests.gradref import bucket_lists, check_gradient

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHORT = list(range(14))
LONG = [62, 63, 64, 65, 66, 67, 255, 256, 257, 258, 319, 320, 321, 511, 512, 513]


@pytest.mark.parametrize("T,D,L,k,sizes", [
    (300, 1030, 1, 1, SHORT),         # direct, 0 or 1 forward terms
    (300, 5, 1, 3, SHORT),            # direct and listed, 0 or 3
    (700, 260, 1, 9, SHORT + LONG),   # forward terms alone beyond the direct ones
    (700, 6, 4, 12, SHORT + LONG),    # several buckets a row
    (1400, 1025, 16, 6, SHORT + LONG),
])
def test_rows_by_number_of_terms(T, D, L, k, sizes):
    print(f"[gpu] gradient rows T={T} D={D} L={L} k={k}", flush=True)
    rng = np.random.default_rng(T + D)
    n = T - L + 1
    w = rng.standard_normal(n)
    w[rng.permutation(n)[:n // 5]] = 0.0
    step = n // len(sizes)
    assert step >= 2 * L
    idx = bucket_lists(rng, n, k, w, sizes, step * np.arange(len(sizes)))
    idx[(idx == -1) & (rng.random(idx.shape) < 0.5)] = n  # not a trajectory either
    check_gradient(T, D, L, k, idx, w, T)
