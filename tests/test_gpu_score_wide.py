"""Score-function gradient at the widths above 16, where a slice's rows are taken four at a time: one
to four rows in the last group, one slice and several, partly filled wavefronts, both leads."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import score as SC  # noqa: E402
from test_gpu_parity import case, gpu_build, oracle_solve  # noqa: E402
from test_gpu_score import gpu_counts, grad_mc  # noqa: E402
from test_gpu_walker import oracle_alias_tables  # noqa: E402


@pytest.mark.parametrize("inject", [0, 1])
@pytest.mark.parametrize("W,L", [(18, 4), (19, 1), (20, 4), (21, 3), (22, 2), (23, 3), (24, 1),
                                 (26, 3), (28, 2), (30, 3), (32, 2)])
def test_gradient_equals_the_oracle(W, L, inject):
    c = case(W=W, L=L, eta=0.25, disorder=0.3, nE=2, emin=-1.4, emax=1.2, seed=W + L)
    k = gpu_build(c)
    thr, al = oracle_alias_tables(oracle_solve(c), k.alias_pitch)
    k.set_alias_tables(thr, al)
    nw = 5_000
    cnt, tal = gpu_counts(k, nw, inject)
    dV, dG = grad_mc(k, cnt, tal, c["w"], inject)
    n = k.n_out
    rc = cnt.cpu().numpy().view(np.uint32).reshape(2, n, n).astype(np.int64)
    rV, rG = np.zeros(W * L), np.zeros(W * L)
    for e, (E, w) in enumerate(zip(c["E"], c["w"])):
        v, g = SC.score_gradient(W, L, 1.0, c["V"], c["g"], E, rc[e], nw, inject)
        rV += w * v
        rG += w * g
    # the bound of the gradients on wires up to W = 32
    assert np.abs(dV - rV).max() <= 1e-9 * np.abs(rV).max()
    assert np.abs(dG - rG).max() <= 1e-9 * np.abs(rG).max()
