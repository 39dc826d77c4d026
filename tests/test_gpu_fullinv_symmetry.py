"""The lower half of G and its transposed copies: ragged last column tiles, slices across the
128-byte lines of the transposed rows, single slices, and the exit weights of the first slice."""
import numpy as np
import pytest
import torch

from oracle import dense as D
from paper_1805_10164_amd import inputs
from paper_1805_10164_amd import mcnegf as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,L", [(1, 1), (1, 64), (1, 131), (2, 40), (3, 22), (5, 13), (5, 39),
                                 (6, 1), (7, 19), (8, 17), (9, 15), (11, 12), (13, 5), (14, 10),
                                 (16, 1), (16, 9), (17, 8), (21, 7), (27, 5), (31, 3), (32, 1),
                                 (32, 9)])
def test_rows_symmetric_and_equal_to_dense(W, L):
    dev = "cuda"
    N, nE = W * L, 9  # one more energy than there are XCDs
    V = inputs.random_sites(N, 3 * W + L, -0.5, 0.5)
    g = inputs.random_sites(N, 5 * W + L, 0.01, 0.2)
    E, _ = inputs.energy_grid(-1.6, 1.7, nE)
    put = lambda x: torch.tensor(x, dtype=torch.float64, device=dev)
    sysm = M.make_system(W, L, flags=M.BUILD_NO_ALIAS | M.BUILD_NO_DIRECT)
    ws = M.allocate_workspace(sysm, nE, dev)
    ws.view(torch.uint8).fill_(0xFF)  # NaN wherever an entry is not written
    tV, tg, tE = put(V), put(g), put(E)
    k = M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    assert M.mc_negf_status(k) == 0
    P = k.P().cpu().numpy()
    wL, wR = k.wL().cpu().numpy(), k.wR().cpu().numpy()
    assert np.isfinite(P).all()
    for e in (0, 4, 8):
        # the transposed copy is the same number, except inside the diagonal blocks, which are
        # inverted as a whole
        for x in range(L):
            s = slice(x * W, (x + 1) * W)
            P[e][s, s] = 0.5 * (P[e][s, s] + P[e][s, s].T)
        assert np.array_equal(P[e], P[e].T)
        SL = D.lead_self_energy(E[e], W, 1.0)
        G = D.retarded_green(E[e], D.hamiltonian(W, L, 1.0, V), W, L, SL, SL, g)
        S = D.broadening(SL).real
        A = np.abs(G) ** 2
        # parity tolerances of the build: relative to the largest entry of the row
        assert (np.abs(P[e] - A).max(axis=1) <= 1e-10 * A.max(axis=1)).all()
        for w, rows in ((wL[e], G[:W]), (wR[e], G[N - W:])):
            ref = np.einsum("aj,ab,bj->j", rows.conj(), S, rows).real
            assert np.abs(w - ref).max() <= 1e-10 * ref.max()
