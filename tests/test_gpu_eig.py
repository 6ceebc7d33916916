"""The projected eigenproblem (GPU) where its kernels change: matrices around 64 and 128 rows (two instances of one workgroup, or several),
more than 255 wanted values (a workgroup or 32 threads for each), a single vector, the smallest sizes."""
import numpy as np
import pytest

from gpu_common import pair, say
from workloads import SD_ORBITS, SD_SPE, random_tbme

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# nb, n_eig, l_s, l_m: the matrix reaches l_m - nb rows
CASES = [(1, 1, 1, 3), (1, 3, 8, 65), (1, 3, 8, 66), (1, 3, 8, 128), (1, 3, 8, 129), (1, 3, 8, 130), (2, 6, 40, 131), (4, 10, 20, 132),
         (4, 10, 20, 136), (4, 254, 256, 320), (4, 260, 260, 330)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_levels_match_dense(case):
    """Converged to residuals tol * |H| = 1e-9 |H|: eigenvalues within the residual norm of the dense ones, far
    inside 1e-8 relative; eigenvectors orthonormal and with those residuals."""
    nb, n, ls, lm = case
    say("case", case)
    g, o = pair(SD_ORBITS, 2, 2, 0, random_tbme(SD_ORBITS, 1), SD_SPE, SD_SPE)
    H = o.dense()
    e = np.linalg.eigvalsh(H)
    ev, X, info = g.solve(nb, n, ls, lm, 1e-9, vectors=True, max_iter=20000)
    assert info.converged
    norm = np.abs(e).max()
    assert np.all(np.abs(ev - e[:n]) <= 1e-8 * norm)
    x = X.cpu().numpy()
    assert np.abs(x.T @ x - np.eye(n)).max() <= 1e-10
    assert np.linalg.norm(H @ x - x * ev, axis=0).max() <= 2e-8 * norm
