"""The dense steps of a solve (GPU) where their kernels change: block widths around 4, 8 and 16 (one element of the
Cholesky factor a thread, the partial sums in its launch or not), few and many row chunks, ragged basis widths."""
import numpy as np
import pytest

from gpu_common import pair, say
from workloads import SD_ORBITS, SD_SPE, random_tbme

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [1, 2, 4, 5, 8, 9, 16, 17, 33])
def test_block_widths_match_dense(nb):
    """sd 2+2 (D = 640): converged to residuals 1e-9 |H|, so eigenvalues within 1e-8 |H| of the dense ones;
    eigenvectors orthonormal to the rounding of the basis."""
    g, o = pair(SD_ORBITS, 2, 2, 0, random_tbme(SD_ORBITS, 1), SD_SPE, SD_SPE)
    H = o.dense()
    e = np.linalg.eigvalsh(H)
    n = 3
    ev, X, info = g.solve(nb, n, 10, 60 + 5 * nb, 1e-9, vectors=True, max_iter=20000)
    say("nb", nb, "iterations", info.iterations)
    assert info.converged
    norm = np.abs(e).max()
    assert np.all(np.abs(ev - e[:n]) <= 1e-8 * norm)
    x = X.cpu().numpy()
    assert np.abs(x.T @ x - np.eye(n)).max() <= 1e-10
    assert np.linalg.norm(H @ x - x * ev, axis=0).max() <= 2e-8 * norm
