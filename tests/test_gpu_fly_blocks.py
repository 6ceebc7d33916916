"""Single-species pair blocks (GPU) where their kernels change: blocks of up to 16, 32 and 64 pairs, no, one or
two spectators, and widths around one column, one 16-byte lane, a slot row and several column tiles."""
import os

import numpy as np
import pytest

from gpu_common import pair, say, term_bound
from workloads import SD_ORBITS, SNSB_ORBITS, random_block, random_tbme

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ONE_PAR = ((0, 6, 13), (0, 4, 9), (1, 4, 7))   # all of one parity, 32 m-states: blocks of up to 42 pairs
ONE_PAR36 = ((0, 6, 13), (0, 6, 11), (0, 4, 9))  # 36 m-states: up to 50 pairs

CASES = [("sd_n2", SD_ORBITS, 2, 0, 0), ("one_parity_n3", ONE_PAR, 3, 1, 0),
         ("snsb_n4", SNSB_ORBITS, 4, 0, 1)]


def _forced(orbits, n, twoM, spe, par, oracle=True):
    os.environ["TRBL_FLY"] = "1"
    try:
        return pair(orbits, 0, n, twoM, random_tbme(orbits, 31), spe, spe, par, oracle)
    finally:
        del os.environ["TRBL_FLY"]


@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0])
def test_widths_match_dense_oracle(case):
    """Every width against the oracle's explicit H, within the rounding bound of its terms (blocks of at most 64
    pairs, then the C(n, 2) core slots), in FP64 and FP32."""
    name, orbits, n, twoM, par = case
    say("case", name)
    spe = [(-0.8 + 0.5 * k) for k in range(len(orbits))]
    g, o = _forced(orbits, n, twoM, spe, par)
    H = o.dense()
    rows = np.arange(o.dim)
    V = random_block(7, o.dim, 33)
    ref, ref32 = H @ V, H @ V.astype(np.float32).astype(np.float64)
    ex = n * (n - 1) // 2 + 64
    b64 = term_bound(o, rows, V, extra=ex)
    b32 = term_bound(o, rows, V.astype(np.float32), fp32=True, extra=ex)
    for nb in (1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 24, 33):
        W = g.apply(torch.from_numpy(np.ascontiguousarray(V[:, :nb])).cuda()).cpu().numpy()
        assert np.all(np.abs(W - ref[:, :nb]) <= b64[:, :nb]), nb
        W = g.apply(torch.from_numpy(np.ascontiguousarray(V[:, :nb].astype(np.float32))).cuda()).cpu().numpy()
        assert np.all(np.abs(W - ref32[:, :nb]) <= b32[:, :nb]), nb


def test_widest_blocks_match_per_element_kernel():
    """Blocks beyond 48 pairs (more m-states than the oracle takes) against the per-element kernel: a row of three
    nucleons sums at most 3 * 50 products and three energies on either path, below hmax * vmax each."""
    spe = [0.3, -0.2, 0.5]
    g, _ = _forced(ONE_PAR36, 3, 1, spe, 0, oracle=False)
    os.environ["TRBL_PN_TILES"] = "0"
    try:
        g0, _ = _forced(ONE_PAR36, 3, 1, spe, 0, oracle=False)
    finally:
        del os.environ["TRBL_PN_TILES"]
    say("widest blocks, D", g.dim)
    hmax = float(np.abs(np.array([t[-1] for t in random_tbme(ONE_PAR36, 31)])).max()) * 4 + 3
    V = random_block(8, g.dim, 16)
    terms = 160
    for dt, u in ((torch.float64, 2.0 ** -53), (torch.float32, 2.0 ** -24)):
        for nb in (1, 8, 16):
            x = torch.from_numpy(np.ascontiguousarray(V[:, :nb])).to("cuda", dt)
            d = (g.apply(x) - g0.apply(x)).abs().max().item()
            assert d <= 2 * terms * terms * u * hmax * np.abs(V).max(), (dt, nb)
