"""Monte Carlo current of given tallies at energy counts either side of the sum's 256 threads, on
the host and into device memory, with energies that have no or one walker; and a build clears the
flags that an earlier one left."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1805_10164_amd import mcnegf as M  # noqa: E402


@pytest.mark.parametrize("nE", [1, 2, 255, 256, 257, 1300])
def test_current_of_tallies(nE):
    dev = "cuda"
    put = lambda x: torch.tensor(x, device=dev)
    sysm = M.make_system(1, 2)
    ws = M.allocate_workspace(sysm, nE, dev)
    tV, tg, tE = put(np.zeros(2)), put(np.full(2, 0.1)), put(np.linspace(-1.5, 1.5, nE))
    k = M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    rng = np.random.default_rng(nE)
    tal = np.zeros((nE, M.TALLY_N), dtype=np.int64)
    tal[:, :3] = rng.integers(0, 900, size=(nE, 3))
    tal[nE // 2, :3] = 0
    tal[nE // 3, :3] = (0, 1, 0)
    w = rng.uniform(0.1, 1.0, nE)
    for inject in (0, 1):
        T = torch.empty(nE, dtype=torch.float64, device=dev)
        sg = torch.empty_like(T)
        out = torch.empty(2, dtype=torch.float64, device=dev)
        M.mc_negf_current_async(k, 0, inject, put(tal), put(w), T, sg, out)
        _, I, sI = M.mc_negf_current(k, 0, inject, put(tal), put(w), T, sg)
        c = k.lead().cpu().numpy()[:, M.LEAD_CL if inject == 0 else M.LEAD_CR]
        n = tal[:, :3].sum(axis=1).astype(float)
        p = np.where(n > 0, tal[:, 1 - inject] / np.maximum(n, 1), 0.0)
        Tr = c * p
        sr = np.where(n > 1, c * np.sqrt(p * (1 - p) / np.maximum(n - 1, 1)), 0.0)
        # a few rounded operations per entry, then a sum of nE terms of one sign
        assert (np.abs(T.cpu().numpy() - Tr) <= 4 * 2.0 ** -52 * Tr).all()
        assert (np.abs(sg.cpu().numpy() - sr) <= 16 * 2.0 ** -52 * sr).all()
        Ir, sIr = float((w * Tr).sum()), float(np.sqrt((w * w * sr * sr).sum()))
        assert abs(I - Ir) <= (nE + 8) * 2.0 ** -52 * Ir
        assert abs(sI - sIr) <= (nE + 32) * 2.0 ** -52 * sIr
        assert out.cpu().tolist() == [I, sI]
    # walks cut at one step set a flag; the next build starts without flags
    M.mc_negf_walk(k, 1, 0, 0, 0, 2000, 1, torch.zeros_like(put(tal)))
    assert M.mc_negf_status(k) & M.FLAG_TRUNC
    M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    assert M.mc_negf_status(k) == 0
