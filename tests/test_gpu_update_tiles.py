"""The 128 x 128 update tiles of the DIRECT factorization with a ragged last tile column: the padded
size is no multiple of 128, the bordered rows share the last tile row with the matrix's."""
import numpy as np
import pytest
import torch

from paper_1805_10164_amd import inputs
from paper_1805_10164_amd import mcnegf as M

pytestmark = pytest.mark.gpu


def tile_choices(N, nE, cus):
    """(panels of the update, columns, whether its tiles are 128 x 128) of every update."""
    Np = (N + 15) // 16 * 16
    out = []
    for J in range(1, (Np + 127) // 128 - 1, 2):
        m = (J + 1) & -(J + 1)
        c1 = (J + 1) * 128
        wide = min(128 * m, Np - c1)

        def tiles(side):
            nct, nrt = -(-wide // side), -(-(Np + 2 - c1) // side)
            return nct * (nct + 1) // 2 + (nrt - nct) * nct
        big = m >= 8 and tiles(128) * nE >= cus and 100 * tiles(128) <= 26 * tiles(64)
        out.append((m, wide, big))
    return out


@pytest.mark.parametrize("W,L", [(16, 255), (11, 370)])
def test_ragged_large_tiles(W, L):
    dev = "cuda"
    N, nE = W * L, 2
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert any(big and wide % 128 for _, wide, big in tile_choices(N, nE, cus))
    V = inputs.random_sites(N, 11 * W + L, -0.3, 0.3)
    g = inputs.random_sites(N, 7 * W + L, 0.02, 0.12)
    E, w = inputs.energy_grid(-0.9, 1.1, nE)
    put = lambda x: torch.tensor(x, dtype=torch.float64, device=dev)
    sysm = M.make_system(W, L, flags=M.BUILD_NO_ALIAS)
    ws = M.allocate_workspace(sysm, nE, dev)
    tV, tg, tE, tw = put(V), put(g), put(E), put(w)
    k = M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    T = torch.full((2, nE), float("nan"), dtype=torch.float64, device=dev)
    sig = torch.empty(nE, dtype=torch.float64, device=dev)
    for p in (0, 1):
        assert M.mc_negf_current(k, 1, p, None, tw, T[p], sig)[0] == M.OK
    T = T.cpu().numpy()
    wL, wR, A = (x.cpu().numpy() for x in (k.wL(), k.wR(), k.Adiag()))
    lead = k.lead().cpu().numpy()
    P = k.P()[0].cpu().numpy()
    # gamma_j A_jj n_j - sum_i gamma_j gamma_i |G_ji|^2 n_i = gamma_j w_L(j) from the built rows
    Mx = np.diag(g * A[0]) - g[:, None] * g[None, :] * P
    n = np.linalg.solve(Mx, g * wL[0])
    ref = lead[0, M.LEAD_TRL] + float((g * wR[0]) @ n)
    # the parity tolerance of the DIRECT transmissions; T_RL = T_LR by reciprocity
    assert abs(T[0, 0] - ref) <= 1e-10 * ref
    assert (np.abs(T[0] - T[1]) <= 1e-10 * T[0]).all()
