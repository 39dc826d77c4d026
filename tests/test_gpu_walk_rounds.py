"""Walks over energies on either side of a launch: 128 of small tables, 32 of large ones, with a
last launch of a few.  The counting walker, one launch over all energies, walks the same paths."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1805_10164_amd import mcnegf as M  # noqa: E402
from test_gpu_parity import DEV, SEED, case, gpu_build  # noqa: E402
from test_gpu_score import gpu_counts  # noqa: E402


@pytest.mark.parametrize("W,L,nE", [(1, 5, 7), (1, 5, 8), (2, 4, 33), (1, 5, 127), (1, 5, 128),
                                    (2, 4, 129), (1, 3, 256), (1, 3, 261), (4, 96, 42)])
def test_tallies_do_not_depend_on_the_rounds(W, L, nE):
    c = case(W=W, L=L, eta=0.3, disorder=0.3, nE=nE, emin=-1.5, emax=1.5)
    k = gpu_build(c)
    for inject in (0, 1):
        _, ref = gpu_counts(k, 700, inject, begin=5)
        tal = torch.zeros((nE, M.TALLY_N), dtype=torch.int64, device=DEV)
        M.mc_negf_walk(k, SEED, 0, inject, 5, 700, 1_000_000, tal)
        torch.cuda.synchronize()
        assert (tal.cpu().numpy() == ref.cpu().numpy()).all()
        assert (tal.cpu().numpy()[:, :3].sum(axis=1) == np.int64(700)).all()
