"""The DIRECT probe solve at the sizes where its blocked factorization changes shape: one
16-column sub-block, partial and full panels of 128 columns, an odd or even number of panels,
ragged last panels, and enough energies for the large update tiles."""
import numpy as np
import pytest
import torch

from oracle import dense as D
from paper_1805_10164_amd import inputs
from paper_1805_10164_amd import mcnegf as M

pytestmark = pytest.mark.gpu

# (W, L, energies): N + padding = 16, 16, 32, 112, 128, 128, 144, 256, 272, 384, 400, 528, 656,
# 896; 400 and 528 with many energies; 3568, whose update of eight panels has 128 x 128 tiles
CASES = [(3, 5, 2), (2, 8, 2), (1, 17, 2), (2, 56, 2), (1, 127, 2), (4, 32, 2), (3, 43, 2),
         (8, 32, 2), (1, 257, 2), (6, 64, 2), (5, 79, 3), (3, 171, 2), (16, 41, 2), (7, 128, 2),
         (4, 100, 96), (11, 48, 61), (16, 223, 2)]


@pytest.mark.parametrize("W,L,nE", CASES)
def test_direct_current_at_panel_edges(W, L, nE):
    dev = "cuda"
    N = W * L
    V = inputs.random_sites(N, 11 * W + L, -0.4, 0.4)
    g = inputs.random_sites(N, 7 * W + L, 0.02, 0.12)
    g[inputs.random_sites(N, 5, 0.0, 1.0) < 0.1] = 0.0  # probes without dephasing: identity rows
    E, w = inputs.energy_grid(-1.7, 1.6, nE)
    put = lambda x: torch.tensor(x, dtype=torch.float64, device=dev)
    sysm = M.make_system(W, L, flags=M.BUILD_NO_ALIAS)
    ws = M.allocate_workspace(sysm, nE, dev)
    tV, tg, tE, tw = put(V), put(g), put(E), put(w)
    k = M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    T = torch.full((2, nE), float("nan"), dtype=torch.float64, device=dev)
    sig = torch.empty(nE, dtype=torch.float64, device=dev)
    I = []
    for p in (0, 1):
        st, cur, _ = M.mc_negf_current(k, 1, p, None, tw, T[p], sig)
        assert st == M.OK
        I.append(cur)
    T = T.cpu().numpy()
    pick = sorted({0, nE // 2, nE - 1})
    ref = np.array([s.T_eff for s in D.solve_workload(W, L, 1.0, V, g, E[pick])])
    # the parity tolerance of the DIRECT transmissions: backward-stable FP64 solves of systems
    # whose condition is below 1e4 agree to well under 1e-10; T_RL = T_LR by reciprocity
    for p in (0, 1):
        assert np.abs(T[p][pick] - ref).max() <= 1e-10 * max(ref.max(), 1e-3)
        assert abs(I[p] - float((w * T[p]).sum())) <= 1e-12 * abs(I[p]) + 1e-15
