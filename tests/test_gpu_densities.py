"""Gradient densities (GPU) at the edges of their tiles: numbers of vectors around the lanes of a row, pair blocks
of more than 16 and 32 pairs, one particle of a species, both parities; against the oracle."""
import numpy as np
import pytest

from gpu_common import pair, say
from oracle.grad import spe_gradient, tbme_gradient
from workloads import PF_ORBITS, SD_ORBITS, grad_weights, random_block, random_tbme

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIXED_PAR = ((0, 1, 1), (0, 2, 5), (0, 1, 3))
SPACES = {
    "sd22": (SD_ORBITS, 2, 2, 0, 0),
    "pf21": (PF_ORBITS, 2, 1, 1, 0),  # pn blocks of up to 60 pairs, pp blocks of up to 30
    "mixpar": (MIXED_PAR, 2, 3, 1, -1),
    "protons": (SD_ORBITS, 4, 0, 0, 0),
}


@pytest.mark.parametrize("space", SPACES)
@pytest.mark.parametrize("n", [1, 2, 3, 5, 8, 24, 25])
def test_densities_match_oracle(space, n):
    """Both sides are sums over D x n products x_i h x_j; the oracle forms H' x row by row, so the two differ by
    rounding of at most (number of products + moves per row) units of sum w |x| |H'| |x|, bounded here
    by |x|^2 times the largest row sum of |H'|: at most 64 unit elements a row times the coefficients (<= 2)."""
    orbits, z, nn, twoM, par = SPACES[space]
    say("case", space, n)
    tb = random_tbme(orbits, 3)
    g, o = pair(orbits, z, nn, twoM, tb, [0.0] * len(orbits), [0.0] * len(orbits), par)
    X, w = random_block(17, o.dim, n), grad_weights(n)
    gv, gs = g.tbme_grad(w, evecs=torch.from_numpy(X).cuda())
    scale = float(np.sum(w * np.sum(X * X, axis=0))) * 128.0
    tol = 2.0 ** -53 * (o.dim * n + 64) * scale
    assert np.all(np.abs(gv - tbme_gradient(o, tb, X, w)) <= tol)
    assert np.all(np.abs(gs - spe_gradient(o, X, w)) <= tol)
