"""Solves of Hamiltonians in very large and very small units (GPU)."""
import numpy as np
import pytest

from gpu_common import say
from workloads import SD_ORBITS, SD_SPE, random_tbme

import paper_1902_02064_amd as trbl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [2, 4, 8, 16, 17])
@pytest.mark.parametrize("k", [300, -300])
def test_solve_scales_with_the_units(nb, k):
    """H times 2^k: every sum, product, quotient and square root of the FP64 solve scales by a power of two (block
    norms by 2^k, Gram matrices by 2^2k, all far inside the range of a double), and every test compares scaled
    numbers. So the run takes the same iterations and gives the same bits times 2^k."""
    tb = random_tbme(SD_ORBITS, 1)
    run = []
    for f in (1.0, 2.0 ** k):
        g = trbl.Model(SD_ORBITS, 2, 2, 0)
        spe = [f * e for e in SD_SPE]
        g.set_hamiltonian(spe, spe, [t[:6] + (f * t[6],) for t in tb])
        ev, _, info = g.solve(nb, 4, 12, 12 + 10 * nb, 1e-9)
        say("nb", nb, "factor", f, "iterations", info.iterations)
        assert info.converged
        run.append((ev / f, info.iterations))
    assert run[0][1] == run[1][1]
    assert np.array_equal(run[0][0], run[1][0])
