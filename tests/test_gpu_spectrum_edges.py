"""Energy-resolved current from given tallies and histograms, at energy counts on either side of
the kernel's groups of 16 entries and 16 partial sums, with energies that no walker started at."""
import numpy as np
import pytest
import torch

from oracle import inelastic as IN
from paper_1805_10164_amd import mcnegf as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inject", [0, 1])
@pytest.mark.parametrize("nE", [1, 2, 15, 16, 17, 33, 250])
def test_spectrum_equals_the_oracle(nE, inject):
    dev = "cuda"
    put = lambda x: torch.tensor(x, device=dev)
    sysm = M.make_system(2, 3, flags=M.BUILD_NO_DIRECT)
    ws = M.allocate_workspace(sysm, nE, dev)
    V, g, E = np.zeros(6), np.full(6, 0.1), np.linspace(-1.5, 1.5, nE)
    k = M.mc_negf_build_kernel(sysm, put(V), put(g), put(E), ws)
    rng = np.random.default_rng(nE)
    tal = rng.integers(0, 1000, size=(nE, M.TALLY_N)).astype(np.int64)
    tal[nE // 2:nE // 2 + 1] = 0  # no walkers there
    hist = rng.integers(0, 3, size=(2, nE, nE)).astype(np.int64)
    w = rng.uniform(0.1, 1.0, nE)
    S = torch.full((2, nE), 7.0, dtype=torch.float64, device=dev)
    M.mc_negf_spectrum(k, inject, put(tal), put(hist), put(w), S)
    c = k.lead().cpu().numpy()[:, M.LEAD_CL if inject == 0 else M.LEAD_CR]
    ref = IN.spectrum(tal, hist, c, w, inject)
    # positive terms, each product and quotient rounded, at most nE - 1 additions
    assert (np.abs(S.cpu().numpy() - ref) <= (nE + 8) * 2.0 ** -52 * ref).all()
