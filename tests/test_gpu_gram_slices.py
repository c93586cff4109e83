"""The Gram's K pipeline at its edges: the operands move in slices (16 cells in
FP32 and BF16x3, 32 in FP16), four of them in flight, with a norm correction
every 512 cells. D runs over one pair of slices, the pairs around the pipeline's
depth, and the chunk boundary, each with a ragged neighbour; T over a partial
tile, one past a tile and one past a batch of converted rows.

Every listed distance is compared with the oracle's distance of the same pair,
and every row's k-th with the oracle's k-th, within the precision's tolerance
plus the Gram's norm-relative allowance (Eq. 4 in FP32 accumulation).
"""
import numpy as np
import pytest

import oracle
from paper_2603_02059_amd import synth
from tests.parity import gram_norm_tol, precision_tol, snapshot_norms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,rb", [(700, 304), (2300, 512), (2561, 1024), (6400, 1536)])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "fp16"])
def test_tile_sizes_agree(T, rb, prec):
    """The whole matrix and the passes of band mode take different Gram tiles
    (256, 128 or 64 fields, by how many the launch has), so equal lists mean
    equal distances from every shape, ragged last tiles and rows included."""
    from paper_2603_02059_amd import traknn as tk
    D, L, k = 77, 4, 6
    print(f"[gpu] tiles T={T} row_batch={rb} {prec}", flush=True)
    X = torch.from_numpy(synth.make_fields(T, 7, 11, sigma=1.0, n_events=2, event_len=L,
                                           seed=T)[0]).cuda()
    a, b = tk.knn(X, L, k, prec), tk.knn(X, L, k, prec, row_batch=rb)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "fp16"])
@pytest.mark.parametrize("T,D", [(257, 32), (257, 33), (261, 64), (262, 65), (256, 96), (300, 129),
                                 (300, 511), (300, 512), (300, 513), (513, 545), (300, 1056),
                                 (2300, 33), (2049, 129)])
def test_gram_slice_edges(T, D, prec):
    from paper_2603_02059_amd import traknn as tk
    L, k = 3, 5
    print(f"[gpu] slices T={T} D={D} {prec}", flush=True)
    Xn, _ = synth.make_fields(T, 1, D, sigma=2.0, n_events=1, event_len=L, seed=T + D)
    X = torch.from_numpy(Xn).cuda()
    idx, dist = tk.knn(X, L, k, prec)
    idx, dist = idx[0].cpu().numpy(), dist[0].cpu().numpy()
    n = T - L + 1
    Dm = oracle.traj_dist(Xn, L)
    ref = np.take_along_axis(Dm, idx, axis=1)
    N = snapshot_norms(Xn)
    Nt = sum(N[m:m + n] for m in range(L))
    allow = precision_tol(prec) * ref + gram_norm_tol(prec, D) * (Nt[:, None] + Nt[idx])
    assert np.all(np.abs(idx - np.arange(n)[:, None]) >= L)
    assert np.all(np.abs(dist - ref) <= allow)
    kth = oracle.knn(Xn, L, k)[1][:, -1]
    assert np.all(ref[:, -1] <= kth + 2 * allow.max(axis=1))
