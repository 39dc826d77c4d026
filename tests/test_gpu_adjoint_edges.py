"""The adjoint at the edges of its column tiles: one slice, partly filled tiles of 32 and 64
columns, both injection leads, and every kind of block width (VALU, matrix cores)."""
import numpy as np
import pytest
import torch

from oracle import grad as OG
from paper_1805_10164_amd import inputs
from paper_1805_10164_amd import mcnegf as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inject", [0, 1])
@pytest.mark.parametrize("W,L", [(1, 1), (1, 33), (2, 16), (3, 11), (8, 5), (9, 7), (15, 3),
                                 (16, 1), (16, 2), (16, 5), (17, 3), (24, 2), (31, 2), (32, 1),
                                 (32, 3)])
def test_gradient_equals_dense_adjoint(W, L, inject):
    dev = "cuda"
    N, nE = W * L, 2
    V = inputs.random_sites(N, 13 * W + L, -0.4, 0.4)
    g = inputs.random_sites(N, 19 * W + L, 0.02, 0.15)
    E, w = inputs.energy_grid(-1.3, 1.1, nE)
    put = lambda x: torch.tensor(x, dtype=torch.float64, device=dev)
    sysm = M.make_system(W, L, flags=M.BUILD_NO_ALIAS)
    ws = M.allocate_workspace(sysm, nE, dev)
    tV, tg, tE, tw = put(V), put(g), put(E), put(w)
    k = M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    gws = torch.empty(M.mc_negf_grad_workspace_bytes(k), dtype=torch.uint8, device=dev)
    dV, dg = torch.empty_like(tV), torch.empty_like(tg)
    st, I = M.mc_negf_grad(k, inject, tw, gws, dV, dg)
    assert st == M.OK
    # T_LR = T_RL, so one dense derivative serves both leads
    I_ref, dV_ref, dg_ref = OG.adjoint(W, L, 1.0, V, g, E, w)
    assert abs(I - I_ref) <= 1e-10 * abs(I_ref)
    # the gradient's parity tolerance: 1e-9 of the largest derivative
    for got, ref in ((dV, dV_ref), (dg, dg_ref)):
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-9 * max(np.abs(ref).max(), 1e-6)
