"""Monte Carlo current of given tallies at energy counts on either side of the change from one
workgroup to the whole chip, and at 70000 energies: entries, sums, and the sums in device memory."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1805_10164_amd import mcnegf as M  # noqa: E402


@pytest.mark.parametrize("nE", [8191, 8192, 8193, 70_000])
def test_current_of_many_tallies(nE):
    dev = "cuda"
    put = lambda x: torch.tensor(x, device=dev)
    sysm = M.make_system(1, 1)
    ws = M.allocate_workspace(sysm, nE, dev)
    tV, tg, tE = put(np.zeros(1)), put(np.full(1, 0.1)), put(np.linspace(-1.5, 1.5, nE))
    k = M.mc_negf_build_kernel(sysm, tV, tg, tE, ws)
    rng = np.random.default_rng(nE)
    tal = np.zeros((nE, M.TALLY_N), dtype=np.int64)
    tal[:, :3] = rng.integers(0, 900, size=(nE, 3))
    tal[nE // 2, :3] = 0
    tal[nE - 1, :3] = (0, 1, 0)
    w = rng.uniform(0.1, 1.0, nE)
    T = torch.empty(nE, dtype=torch.float64, device=dev)
    sg = torch.empty_like(T)
    out = torch.empty(2, dtype=torch.float64, device=dev)
    with M.LaunchTimes() as lt:
        M.mc_negf_current_async(k, 0, 1, put(tal), put(w), T, sg, out)
    # one workgroup's chain of nE / 256 divisions and square roots is longer than a launch
    assert lt.count("current_sum_kernel") == (nE > 8192)
    _, I, sI = M.mc_negf_current(k, 0, 1, put(tal), put(w), T, sg)
    c = k.lead().cpu().numpy()[:, M.LEAD_CR]
    n = tal[:, :3].sum(axis=1).astype(float)
    p = np.where(n > 0, tal[:, 0] / np.maximum(n, 1), 0.0)
    Tr = c * p
    sr = np.where(n > 1, c * np.sqrt(p * (1 - p) / np.maximum(n - 1, 1)), 0.0)
    # a few rounded operations per entry, then a sum of nE terms of one sign
    assert (np.abs(T.cpu().numpy() - Tr) <= 4 * 2.0 ** -52 * Tr).all()
    assert (np.abs(sg.cpu().numpy() - sr) <= 16 * 2.0 ** -52 * sr).all()
    Ir, sIr = float((w * Tr).sum()), float(np.sqrt((w * w * sr * sr).sum()))
    assert abs(I - Ir) <= (nE + 8) * 2.0 ** -52 * Ir
    assert abs(sI - sIr) <= (nE + 32) * 2.0 ** -52 * sIr
    assert out.cpu().tolist() == [I, sI]
