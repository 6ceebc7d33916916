"""Gradients of nearly full shells (GPU): few states, but far more subsets of the m-states than states."""
import numpy as np
import pytest

from gpu_common import pair, say
from oracle.grad import spe_gradient, tbme_gradient
from workloads import SD_ORBITS, SNSB_ORBITS, grad_weights, random_block, random_tbme

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("space", [(2, 10), (1, 9), (11, 1), (11, 10), (0, 9), (12, 2)], ids=str)
def test_hole_nuclei_match_oracle(space):
    """Both sides are sums over D x n products x_i h x_j: at most (number of products + moves per row) roundings of
    sum w |x|^2 times the largest row sum of |H'| (64 unit elements a row times coefficients of at most 2)."""
    z, n = space
    say("case", space)
    tb = random_tbme(SD_ORBITS, 3)
    g, o = pair(SD_ORBITS, z, n, (z + n) % 2, tb, [0.0] * 3, [0.0] * 3)
    X, w = random_block(17, o.dim, 3), grad_weights(3)
    gv, gs = g.tbme_grad(w, evecs=torch.from_numpy(X).cuda())
    tol = 2.0 ** -53 * (o.dim * 3 + 64) * float(np.sum(w * np.sum(X * X, axis=0))) * 128.0
    assert np.all(np.abs(gv - tbme_gradient(o, tb, X, w)) <= tol)
    assert np.all(np.abs(gs - spe_gradient(o, X, w)) <= tol)


def test_tables_grow_with_the_states():
    """28 protons in the 32 m-states of the 50-82 shell: at most 1,504 states, C(28, 2) pairs of 8 bytes each and as
    many work items of 16 bytes, so 14 MB of tables; with the smaller ones and the allocator's rounding below
    64 MiB. (All subsets of 26 states times all pairs would be 1.8 GB.)"""
    g, _ = pair(SNSB_ORBITS, 28, 0, 0, random_tbme(SNSB_ORBITS, 3), [0.0] * 5, [0.0] * 5, 1, oracle=False)
    assert g.dim <= 1504
    X = torch.from_numpy(random_block(5, g.dim, 2)).cuda()
    g.apply(X)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    gv, gs = g.tbme_grad([1.0, 0.5], evecs=X)
    used = free - torch.cuda.mem_get_info()[0]
    say("states", g.dim, "bytes kept", used)
    assert used <= 64 << 20
    # 28 protons in every state: the occupations add up to 28 sum w |x|^2
    norm = float((X * X).sum(0) @ torch.tensor([1.0, 0.5], dtype=torch.float64, device="cuda"))
    assert abs(gs[:5].sum() - 28 * norm) <= 2.0 ** -53 * (2 * g.dim * 32) * 28 * norm
