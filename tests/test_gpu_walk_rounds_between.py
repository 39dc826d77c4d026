"""Walks whose launches take 5 to 15 energies per XCD, by the size of the tables, with a last launch
of one energy or a few.  The counting walker, one launch over all energies, walks the same paths."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1805_10164_amd import mcnegf as M  # noqa: E402
from test_gpu_parity import DEV, SEED, case, gpu_build  # noqa: E402
from test_gpu_score import gpu_counts  # noqa: E402


# 302, 252 and 202 outcomes: 40, 64 and 96 energies a launch
@pytest.mark.parametrize("W,L,per_launch", [(3, 100, 40), (5, 50, 64), (4, 50, 96)])
@pytest.mark.parametrize("more", [0, 1, 11])
def test_tallies_do_not_depend_on_the_rounds(W, L, per_launch, more):
    nE = per_launch + more
    c = case(W=W, L=L, eta=0.3, disorder=0.3, nE=nE, emin=-1.5, emax=1.5)
    k = gpu_build(c)
    tal = torch.zeros((nE, M.TALLY_N), dtype=torch.int64, device=DEV)
    with M.LaunchTimes() as lt:
        M.mc_negf_walk(k, SEED, 0, 0, 5, 700, 1_000_000, tal)
    assert lt.count("walk_kernel") == (1 if more == 0 else 2)
    _, ref = gpu_counts(k, 700, 0, begin=5)
    assert torch.equal(tal, ref) and bool((tal[:, :3].sum(dim=1) == 700).all())
