"""Alias tables at the row lengths where the threads and items per row change: the smallest rows,
each count of items per thread, and one outcome either side of a change of threads.  The tables
must sample the kernel rows to the thresholds' resolution."""
import numpy as np
import pytest
import torch

from paper_1805_10164_amd import inputs
from paper_1805_10164_amd import mcnegf as M

pytestmark = pytest.mark.gpu

# outcomes N + 2 = 3, 8, 128, 129, 256, 257, 386, 513, 641, 769, 897, 1024, 1025, 1281, 1536,
# 1537, 2050, 2562, 3074, 3586, 4096, 4097, 5122, 6146, 7169, 8192, 8193, 10241, 12290
CASES = [(1, 1), (2, 3), (2, 63), (1, 127), (2, 127), (3, 85), (4, 96), (7, 73), (9, 71), (13, 59),
         (5, 179), (2, 511), (11, 93), (1, 1279), (2, 767), (5, 307), (16, 128), (16, 160),
         (16, 192), (16, 224), (2, 2047), (15, 273), (16, 320), (24, 256), (1, 7167),
         (10, 819), (1, 8191), (1, 10239), (32, 384)]


@pytest.mark.parametrize("W,L", CASES)
def test_tables_sample_the_rows(W, L):
    dev = "cuda"
    N = W * L
    n = N + 2
    V = inputs.random_sites(N, W + 3 * L, -0.3, 0.3)
    g = inputs.random_sites(N, 2 * W + L, 0.02, 0.2)
    E = np.array([0.37])
    put = lambda x: torch.tensor(x, dtype=torch.float64, device=dev)
    sysm = M.make_system(W, L, flags=M.BUILD_NO_DIRECT)
    ws = M.allocate_workspace(sysm, 1, dev)
    tV, tg, tE = put(V), put(g), put(E)
    k = M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    assert M.mc_negf_status(k) == 0
    P = k.P()[0]
    wL, wR = k.wL()[0].cpu().numpy(), k.wR()[0].cpu().numpy()
    rows = sorted({0, N // 3, N - 1})
    thr, alias = k.alias_rows(0, rows)
    for i, r in enumerate(rows):
        w = np.concatenate([g * P[r].cpu().numpy(), [wL[r], wR[r]]])
        assert alias[i].min() >= 0 and alias[i].max() < n
        q = thr[i].astype(np.float64) * 2.0 ** -32
        q[alias[i] == np.arange(n)] = 1.0
        p = q / n
        np.add.at(p, alias[i], (1.0 - q) / n)
        # each bucket's threshold is floored to 2^-32; an outcome collects its own bucket and
        # those aliased to it; the scan's rounding is far below that
        hits = np.bincount(alias[i], minlength=n)
        assert (np.abs(p - w / w.sum()) <= (2.0 + hits) * 2.0 ** -32 / n + 1e-13).all()
