"""DIRECT currents of one to seventeen sites on a handle whose probe vectors have a buffer of their
own, 4 N values per energy and no more: the padded columns read nothing that lies behind it."""
import numpy as np
import pytest
import torch

from oracle import dense as D
from paper_1805_10164_amd import inputs
from paper_1805_10164_amd import mcnegf as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,L", [(1, 1), (1, 2), (2, 1), (1, 3), (1, 4), (5, 1), (3, 5), (1, 17)])
def test_probe_vectors_at_the_end_of_their_buffer(W, L):
    dev = "cuda"
    N, nE = W * L, 3
    V = inputs.random_sites(N, 11 * W + L, -0.4, 0.4)
    g = inputs.random_sites(N, 7 * W + L, 0.05, 0.3)
    E, w = inputs.energy_grid(-1.2, 1.1, nE)
    put = lambda x: torch.tensor(x, dtype=torch.float64, device=dev)
    sysm = M.make_system(W, L, flags=M.BUILD_NO_ALIAS)
    ws = M.allocate_workspace(sysm, nE, dev)
    tV, tg, tE, tw = put(V), put(g), put(E), put(w)
    k = M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    buf = torch.full((64 + nE * 4 * N,), float("nan"), dtype=torch.float64, device=dev)
    k.struct.direct_vec = buf[64:].data_ptr()
    ref = np.array([s.T_eff for s in D.solve_workload(W, L, 1.0, V, g, E)])
    for p in (0, 1):
        T, sig = torch.empty((2, nE), dtype=torch.float64, device=dev)
        st, _, _ = M.mc_negf_current(k, 1, p, None, tw, T, sig)
        assert st == M.OK
        # the parity tolerance of the DIRECT transmissions
        assert np.abs(T.cpu().numpy() - ref).max() <= 1e-10 * ref.max()
